// Bodies into key order (§3.1: the subdivision of space, by Morton keys), for
// systems below kBucketMaxN bodies: the order is that of (key, input index),
// which are all distinct, so it is the one stable order of the keys, however
// it is reached.
//
//   up to kRankMaxN bodies, one launch: every body counts the bodies that
//   come before it (its rank) against keys held in LDS, and goes to its place;
//
//   above, a sample sort: k_splitters ranks a sample of the bodies against
//   itself and keeps every few of them as splitters (the keys of a large
//   sample come from a launch of their own, k_sample_keys), k_bucket_count
//   finds each body's bucket between two splitters, k_bucket_scan and
//   k_bucket_scatter move the bodies with their keys into the buckets, and
//   k_bucket_sort sorts each bucket within LDS and writes its bodies.
//
// Eight passes of an LSD radix sort (each a count, a scan and a scatter of
// the whole array) took 16 to 24 launches of about 5 us at these sizes, and
// its gather then read every body from a random place; here the bodies cross
// memory twice, in 5 or 6 launches.  The scatter carries whole bodies so that
// the second crossing reads them in order (1M bodies: the last kernel took 87
// us when it sorted pairs of key and index and gathered the bodies, 52 so).
// Kernel time from the root cube to the gathered bodies, radix passes / here:
// 1,048,576 bodies 251 / 122 us, 262,144 (2D) 137 / 58, 50,000 108 / 50,
// 10,000 90 / 36, 4,096 (FP64, one launch) 83 / 23.
//
// The sample is drawn at pseudo-random places of equal strata of the input,
// so it follows any input order, and splitters are (key, index) pairs, so
// bodies of equal keys spread over buckets too: a bucket's size depends on
// the draw alone.  A bucket too large for LDS is sorted in memory by one
// block.
#include "tc_internal.h"
#include "keys.h"

namespace tc {
namespace {

using namespace keys;

constexpr int kRankThreads = 1024;
constexpr int kRankOwn = 32;                     // bodies ranked per block
constexpr int kRankChunk = 4096;                 // keys in LDS at a time
constexpr int kBucketCap = 4096;                 // bodies a block sorts in LDS (49 KB: three blocks per CU)
constexpr int kSub = 128;                        // sub-buckets within a bucket
constexpr int kBucketMax = 2048;                 // buckets
constexpr int kSampleFused = 1024;               // samples up to which k_splitters computes the keys itself
constexpr int kFoldTiles = 64;                   // tiles whose counts every scatter block adds up itself

__device__ __forceinline__ int wave_lane() { return threadIdx.x & (kWave - 1); }

// The root cube from a block's boxes, one per thread (1024 threads); block 0
// also stores it.
__device__ __forceinline__ Cube reduce_cube(double (&lo)[3], double (&hi)[3], int bad, int dim, DevParams* prm) {
    __shared__ double s_box[kRankThreads / kWave][6];
    __shared__ int s_bad;
    __shared__ Cube s_cube;
    const int t = threadIdx.x;
    if (t == 0) s_bad = 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fmin(lo[a], __shfl_xor(lo[a], o, kWave));
            hi[a] = fmax(hi[a], __shfl_xor(hi[a], o, kWave));
        }
    }
    __syncthreads();
    if (bad) s_bad = 1;
    if (wave_lane() == 0)
        for (int a = 0; a < 3; ++a) {
            s_box[t / kWave][a] = lo[a];
            s_box[t / kWave][3 + a] = hi[a];
        }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kRankThreads / kWave; ++w)
            for (int a = 0; a < 3; ++a) {
                lo[a] = fmin(lo[a], s_box[w][a]);
                hi[a] = fmax(hi[a], s_box[w][3 + a]);
            }
        s_cube = make_cube(lo, hi, dim);
        if (blockIdx.x == 0) store_cube(s_cube, s_bad != 0, prm);
    }
    __syncthreads();
    return s_cube;
}

// The root cube from the partial boxes of k_bbox_part (7 doubles each), by
// every block for itself.
__device__ __forceinline__ Cube block_cube(const double* __restrict__ part, int nb, int dim, DevParams* prm) {
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int b = threadIdx.x; b < nb; b += kRankThreads) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = fmin(lo[a], part[b * 7 + a]);
            hi[a] = fmax(hi[a], part[b * 7 + 3 + a]);
        }
        bad |= part[b * 7 + 6] != 0.0;
    }
    return reduce_cube(lo, hi, bad, dim, prm);
}

// The same from the bodies themselves, where a block reads them all anyway;
// the masses are checked by the block that stores the cube.
template <typename T, int D>
__device__ __forceinline__ Cube bodies_cube(const T* __restrict__ pos, const T* __restrict__ mass, int n,
                                            DevParams* prm) {
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int i = threadIdx.x; i < n; i += kRankThreads) {
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const double v = (double)pos[(int64_t)i * D + a];
            if (!isfinite(v)) {
                bad = 1;
                continue;
            }
            lo[a] = fmin(lo[a], v);
            hi[a] = fmax(hi[a], v);
        }
        if (blockIdx.x == 0) {
            const double m = (double)mass[i];
            if (!(isfinite(m) && m > 0.0)) bad = 1;
        }
    }
    return reduce_cube(lo, hi, bad, D, prm);
}

template <typename T, int D>
__device__ __forceinline__ uint64_t key_at(const T* __restrict__ pos, int64_t i, const double* lo, double scale) {
    return morton<D>((double)pos[i * D], (double)pos[i * D + 1], D == 3 ? (double)pos[i * D + D - 1] : 0.0, lo, scale);
}

// A body in key order (FP64), and for FP32 inputs a compact copy (exactly
// the input values).
template <typename T>
__device__ __forceinline__ void put_body(T x, T y, T z, T m, int64_t p, Body* __restrict__ bodies,
                                         float4* __restrict__ bodies32) {
    Body b;
    b.x = (double)x;
    b.y = (double)y;
    b.z = (double)z;
    b.m = (double)m;
    bodies[p] = b;
    if (sizeof(T) == 4) bodies32[p] = make_float4((float)x, (float)y, (float)z, (float)m);
}

template <typename T, int D>
__device__ __forceinline__ void put_body_at(const T* __restrict__ pos, const T* __restrict__ mass, int64_t i, int64_t p,
                                            Body* __restrict__ bodies, float4* __restrict__ bodies32) {
    put_body<T>(pos[i * D], pos[i * D + 1], D == 3 ? pos[i * D + D - 1] : T(0), mass[i], p, bodies, bodies32);
}

// How many of the entries e of [e0, e1) come before (key, at), entry e being
// (s_key[e], e).  The block's own entries are [b0, b0 + kRankOwn), so only
// there does the order of the places depend on the lane.
__device__ __forceinline__ uint32_t count_before(const uint64_t* s_key, int e0, int e1, uint64_t key, int at, int b0) {
    uint32_t c = 0;
    const int m0 = max(e0, min(e1, b0)), m1 = max(m0, min(e1, b0 + kRankOwn));
#pragma unroll 8
    for (int e = e0; e < m0; ++e) c += s_key[e] <= key ? 1u : 0u;
    for (int e = m0; e < m1; ++e) c += (s_key[e] < key || (s_key[e] == key && e < at)) ? 1u : 0u;
#pragma unroll 8
    for (int e = m1; e < e1; ++e) c += s_key[e] < key ? 1u : 0u;
    return c;
}

constexpr int kSlices = kRankThreads / kRankOwn;

// One launch for the smallest systems: bound by latency (n <= kRankMaxN: at
// most 256 compares per thread).  Every block computes all keys again, which
// costs less than the launch that would store them, and, without part, the root
// cube, which costs less than the launch of k_bbox_part (a force evaluation of
// 4,096 bodies 93 us with it, 91 without).
template <typename T, int D>
__global__ void __launch_bounds__(kRankThreads) k_rank_sort(const T* __restrict__ pos, const T* __restrict__ mass, int n,
                                                            const double* __restrict__ part, int nb, DevParams* prm,
                                                            uint64_t* __restrict__ keys, uint32_t* __restrict__ perm,
                                                            Body* __restrict__ bodies,
                                                            float4* __restrict__ bodies32) {
    __shared__ uint64_t s_key[kRankChunk];
    __shared__ uint32_t s_rank[kRankOwn];
    const Cube c = part ? block_cube(part, nb, D, prm) : bodies_cube<T, D>(pos, mass, n, prm);
    const int t = threadIdx.x, own = t % kRankOwn, slice = t / kRankOwn;
    const int i0 = (int)blockIdx.x * kRankOwn, i = i0 + own;
    const uint64_t key = i < n ? key_at<T, D>(pos, i, c.lo, c.scale) : 0ull;
    if (t < kRankOwn) s_rank[t] = 0u;
    uint32_t before = 0;
    for (int c0 = 0; c0 < n; c0 += kRankChunk) {
        const int m = min(kRankChunk, n - c0), per = (m + kSlices - 1) / kSlices;
        __syncthreads();
        for (int e = t; e < m; e += kRankThreads) s_key[e] = key_at<T, D>(pos, c0 + e, c.lo, c.scale);
        __syncthreads();
        before += count_before(s_key, min(m, slice * per), min(m, (slice + 1) * per), key, i - c0, i0 - c0);
    }
    atomicAdd(&s_rank[own], before);
    __syncthreads();
    if (t < kRankOwn && i < n) {
        const uint32_t p = s_rank[t];
        keys[p] = key;
        perm[p] = (uint32_t)i;
        put_body_at<T, D>(pos, mass, i, p, bodies, bodies32);
    }
}

// ---------------------------------------------------------- sample sort ----

// A body on its way to its bucket.
template <typename T> struct Rec;
template <> struct __align__(16) Rec<float> {
    uint64_t key;
    uint32_t idx;
    float m, x, y, z, pad;
};
template <> struct __align__(16) Rec<double> {
    uint64_t key;
    uint32_t idx, pad;
    double m, x, y, z;
};

// Place of sample j of S: one in each of S equal strata of the n bodies.
__device__ __forceinline__ int64_t sample_at(int64_t j, int64_t S, int64_t n) {
    const int64_t lo = j * n / S, hi = (j + 1) * n / S;
    uint32_t h = (uint32_t)j * 2654435761u;
    h ^= h >> 15;
    h *= 2246822519u;
    h ^= h >> 13;
    return lo + (int64_t)(h % (uint32_t)(hi - lo));
}

// The keys of a large sample (more than kSampleFused: there every block of
// k_splitters computing all of them costs more than this launch).
template <typename T, int D>
__global__ void __launch_bounds__(kRankThreads) k_sample_keys(const T* __restrict__ pos, int64_t n,
                                                              const double* __restrict__ part, int nb, DevParams* prm,
                                                              int S, uint64_t* __restrict__ out) {
    const Cube c = block_cube(part, nb, D, prm);
    const int j = (int)blockIdx.x * kRankThreads + (int)threadIdx.x;
    if (j < S) out[j] = key_at<T, D>(pos, sample_at(j, S, n), c.lo, c.scale);
}

// Ranks the S samples against each other (their places grow with j, so j
// orders equal keys as the input index does) and keeps the samples of rank
// `per`, 2 per, ... as splitters; the last slot of the B is never less than
// anything.  skeys (nullable): the samples' keys.
template <typename T, int D>
__global__ void __launch_bounds__(kRankThreads) k_splitters(const T* __restrict__ pos, int64_t n,
                                                            const double* __restrict__ part, int nb, DevParams* prm,
                                                            const uint64_t* __restrict__ skeys, int S, int per, int B,
                                                            uint64_t* __restrict__ split_key,
                                                            uint32_t* __restrict__ split_idx) {
    __shared__ uint64_t s_key[kRankChunk];
    __shared__ uint32_t s_rank[kRankOwn];
    Cube c;
    if (!skeys) c = block_cube(part, nb, D, prm);
    const int t = threadIdx.x, own = t % kRankOwn, slice = t / kRankOwn;
    const int j0 = (int)blockIdx.x * kRankOwn, j = min(j0 + own, S - 1);
    const int64_t i = sample_at(j, S, n);
    const uint64_t key = skeys ? skeys[j] : key_at<T, D>(pos, i, c.lo, c.scale);
    if (t < kRankOwn) s_rank[t] = 0u;
    uint32_t before = 0;
    for (int c0 = 0; c0 < S; c0 += kRankChunk) {
        const int m = min(kRankChunk, S - c0), run = (m + kSlices - 1) / kSlices;
        __syncthreads();
        for (int e = t; e < m; e += kRankThreads)
            s_key[e] = skeys ? skeys[c0 + e] : key_at<T, D>(pos, sample_at(c0 + e, S, n), c.lo, c.scale);
        __syncthreads();
        before += count_before(s_key, min(m, slice * run), min(m, (slice + 1) * run), key, j - c0, j0 - c0);
    }
    atomicAdd(&s_rank[own], before);
    __syncthreads();
    if (t < kRankOwn && j0 + t < S) {
        const uint32_t r = s_rank[t];
        if (r > 0 && r % (uint32_t)per == 0) {
            split_key[r / per - 1] = key;
            split_idx[r / per - 1] = (uint32_t)i;
        }
    }
    if (blockIdx.x == 0 && t == 0) {
        split_key[B - 1] = ~0ull;
        split_idx[B - 1] = ~0u;
    }
}

// Splitters of s_k/s_i (B of them, B a power of two) at or before (key, i).
__device__ __forceinline__ int find_bucket(const uint64_t* s_k, const uint32_t* s_i, int B, uint64_t key, uint32_t i) {
    int p = 0;
    for (int step = B >> 1; step > 0; step >>= 1) {
        const uint64_t k = s_k[p + step - 1];
        if (k < key || (k == key && s_i[p + step - 1] <= i)) p += step;
    }
    return p;
}

// Buckets and the tile's count per bucket (hist[tile][bucket]).  A tile is
// PER bodies for each of the block's threads.
template <typename T, int D, int TH, int PER>
__global__ void __launch_bounds__(TH) k_bucket_count(const T* __restrict__ pos, int64_t n,
                                                     const DevParams* __restrict__ prm, int B,
                                                     const uint64_t* __restrict__ split_key,
                                                     const uint32_t* __restrict__ split_idx,
                                                     uint16_t* __restrict__ bucket, uint32_t* __restrict__ hist) {
    __shared__ uint64_t s_k[kBucketMax];
    __shared__ uint32_t s_i[kBucketMax], s_n[kBucketMax];
    const double lo[3] = {prm->lo[0], prm->lo[1], prm->lo[2]}, scale = prm->scale;
    const int t = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * (TH * PER) + t;
    uint64_t key[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) key[q] = key_at<T, D>(pos, min(i0 + TH * q, n - 1), lo, scale);
    for (int b = t; b < B; b += TH) {
        s_k[b] = split_key[b];
        s_i[b] = split_idx[b];
        s_n[b] = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t i = i0 + TH * q;
        if (i >= n) continue;
        const int b = find_bucket(s_k, s_i, B, key[q], (uint32_t)i);
        bucket[i] = (uint16_t)b;
        atomicAdd(&s_n[b], 1u);
    }
    __syncthreads();
    for (int b = t; b < B; b += TH) hist[(int64_t)blockIdx.x * B + b] = s_n[b];
}

// Counts to places within each bucket, over the tiles, and the buckets'
// totals: 32 buckets per block, 32 runs of tiles side by side.
__global__ void __launch_bounds__(1024) k_bucket_scan(uint32_t* __restrict__ hist, int tiles, int B,
                                                      uint32_t* __restrict__ total) {
    __shared__ uint32_t s[32][33];
    const int b = threadIdx.x & 31, run = threadIdx.x >> 5;
    uint32_t* h = hist + (int)blockIdx.x * 32 + b;
    const int per = (tiles + 31) / 32, t0 = run * per, t1 = min(tiles, t0 + per);
    uint32_t sum = 0;
#pragma unroll 8
    for (int t = t0; t < t1; ++t) sum += h[(int64_t)t * B];
    s[run][b] = sum;
    __syncthreads();
    uint32_t at = 0, all = 0;
    for (int r = 0; r < 32; ++r) {
        const uint32_t v = s[r][b];
        if (r < run) at += v;
        all += v;
    }
    for (int t = t0; t < t1; ++t) {
        const uint32_t v = h[(int64_t)t * B];
        h[(int64_t)t * B] = at;
        at += v;
    }
    if (run == 0) total[(int)blockIdx.x * 32 + b] = all;
}

// The bodies into the buckets, in any order within a bucket.  With FOLD
// hist holds the raw counts of a few tiles and each block adds up its own
// places and the totals (cheaper than a launch of k_bucket_scan up to
// kFoldTiles tiles).
template <typename T, int D, int TH, int PER, bool FOLD>
__global__ void __launch_bounds__(TH) k_bucket_scatter(const T* __restrict__ pos, const T* __restrict__ mass, int64_t n,
                                                       const DevParams* __restrict__ prm,
                                                       const uint16_t* __restrict__ bucket, int B,
                                                       const uint32_t* __restrict__ hist, int tiles,
                                                       const uint32_t* __restrict__ total,
                                                       uint32_t* __restrict__ start, Rec<T>* __restrict__ recs) {
    __shared__ uint32_t s_at[kBucketMax];
    __shared__ uint32_t s_w[TH / kWave];
    const double lo[3] = {prm->lo[0], prm->lo[1], prm->lo[2]}, scale = prm->scale;
    const int t = threadIdx.x, lane = wave_lane(), w = t / kWave, tile = (int)blockIdx.x;
    const int64_t i0 = (int64_t)tile * (TH * PER) + t;
    Rec<T> r[PER];
    int b[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int64_t i = min(i0 + TH * q, n - 1);
        r[q].idx = (uint32_t)i;
        r[q].x = pos[i * D];
        r[q].y = pos[i * D + 1];
        r[q].z = D == 3 ? pos[i * D + D - 1] : T(0);
        r[q].m = mass[i];
        r[q].pad = 0;
        b[q] = bucket[i];
    }
    // thread t owns the buckets t * run .. of a run each; their totals'
    // exclusive scan is where each bucket starts
    constexpr int kRun = (kBucketMax + TH - 1) / TH;
    const int run = (B + TH - 1) / TH;
    uint32_t tot[kRun], pre[kRun], sum = 0;
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
        tot[r] = pre[r] = 0u;
        const int bb = t * run + r;
        if (r < run && bb < B) {
            if (FOLD) {
#pragma unroll 8
                for (int q = 0; q < tiles; ++q) {
                    const uint32_t v = hist[(int64_t)q * B + bb];
                    tot[r] += v;
                    if (q < tile) pre[r] += v;
                }
            } else {
                tot[r] = total[bb];
                pre[r] = hist[(int64_t)tile * B + bb];
            }
        }
        sum += tot[r];
    }
    uint32_t x = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) s_w[w] = x;
    __syncthreads();
    uint32_t at = x - sum;
    for (int q = 0; q < w; ++q) at += s_w[q];
#pragma unroll
    for (int r = 0; r < kRun; ++r) {
        const int bb = t * run + r;
        if (r < run && bb < B) {
            s_at[bb] = at + pre[r];
            if (tile == 0) start[bb] = at;
        }
        at += tot[r];
    }
    if (tile == 0 && t == TH - 1) start[B] = (uint32_t)n;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (i0 + TH * q >= n) continue;
        r[q].key = morton<D>((double)r[q].x, (double)r[q].y, (double)r[q].z, lo, scale);
        recs[atomicAdd(&s_at[b[q]], 1u)] = r[q];
    }
}

// One stable counting pass over the digit at `shift`, of the keys or of the
// bodies' indices, in memory by one block: the sort of a bucket too large for
// LDS, as (key, place in the bucket) pairs.
template <typename T, int THREADS>
__device__ void memory_pass(const Rec<T>* __restrict__ recs, const uint64_t* ki, const uint32_t* vi, uint64_t* ko, uint32_t* vo, int m, int shift,
                            bool by_index, uint32_t* s_cnt, uint32_t (*s_wcnt)[256]) {
    const int t = threadIdx.x, lane = wave_lane(), w = t / kWave;
    auto digit = [&](int e) { return by_index ? (recs[vi[e]].idx >> shift) & 255u : (uint32_t)(ki[e] >> shift) & 255u; };
    for (int d = t; d < 256; d += THREADS) s_cnt[d] = 0u;
    __syncthreads();
    for (int e = t; e < m; e += THREADS) atomicAdd(&s_cnt[digit(e)], 1u);
    __syncthreads();
    if (t == 0) {
        uint32_t run = 0;
        for (int d = 0; d < 256; ++d) {
            const uint32_t v = s_cnt[d];
            s_cnt[d] = run;
            run += v;
        }
    }
    __syncthreads();
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    for (int e0 = 0; e0 < m; e0 += THREADS) {
        const int e = e0 + t;
        for (int d = t; d < 256; d += THREADS)
            for (int q = 0; q < THREADS / kWave; ++q) s_wcnt[q][d] = 0u;
        __syncthreads();
        const bool valid = e < m;
        const uint32_t d = valid ? digit(e) : 0u;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        if (valid && before == 0) s_wcnt[w][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        if (valid) {
            uint32_t p = s_cnt[d] + before;
            for (int q = 0; q < w; ++q) p += s_wcnt[q][d];
            ko[p] = ki[e];
            vo[p] = vi[e];
        }
        __syncthreads();
        for (int dd = t; dd < 256; dd += THREADS)
            for (int q = 0; q < THREADS / kWave; ++q) s_cnt[dd] += s_wcnt[q][dd];
        __syncthreads();
    }
}

// Each bucket in order, and its bodies.  A bucket is sorted as the whole was:
// up to kSub of its own keys, ranked, split it into sub-buckets of a few
// keys, and each key counts the ones before it in its sub-bucket.  Keys and
// their places in the bucket stay in LDS (an index is fetched only to order
// equal keys), and the bodies are read again from the bucket, whose lines
// are near.  Bound by the latency of its LDS phases and, at first use, of
// its code, so the loops over a thread's keys are not unrolled (1M bodies:
// 52 us with them unrolled over registers).
template <typename T, int THREADS, int CAP>
__global__ void __launch_bounds__(THREADS) k_bucket_sort(const Rec<T>* __restrict__ recs_all,
                                                         const uint32_t* __restrict__ start, uint64_t* keys_b,
                                                         uint32_t* idx_b, uint64_t* keys_a, uint32_t* idx_a,
                                                         Body* __restrict__ bodies, float4* __restrict__ bodies32) {
    __shared__ uint64_t s_key[CAP];
    __shared__ uint16_t s_ord[CAP];                  // the bucket's places by sub-bucket
    __shared__ uint8_t s_bin[CAP];
    __shared__ uint64_t s_pk[kSub], s_sk[kSub];
    __shared__ uint16_t s_pp[kSub], s_sp[kSub];
    __shared__ uint32_t s_rank[kSub], s_start[kSub + 1], s_next[kSub];
    const int t = threadIdx.x;
    const int64_t s0 = start[blockIdx.x];
    const int m = (int)(start[blockIdx.x + 1] - (uint32_t)s0);
    if (m == 0) return;
    const Rec<T>* recs = recs_all + s0;
    if (m > CAP) {
        // by index, then by key: 12 passes, ending where they began (their
        // counts take the place of the keys in LDS)
        uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_ord);
        uint32_t(*s_wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(s_key);
        static_assert(sizeof(s_key) >= 4 * 256 * (THREADS / kWave) && sizeof(s_ord) >= 4 * 256, "the counts fit");
        uint64_t *ki = keys_b + s0, *ko = keys_a + s0;
        uint32_t *vi = idx_b + s0, *vo = idx_a + s0;
        // the bucket's places stand for the bodies; their indices are read through them
        for (int e = t; e < m; e += THREADS) {
            ki[e] = recs[e].key;
            vi[e] = (uint32_t)e;
        }
        __threadfence_block();
        __syncthreads();
        for (int p = 0; p < 12; ++p) {
            memory_pass<T, THREADS>(recs, ki, vi, ko, vo, m, p < 4 ? 8 * p : 8 * (p - 4), p < 4, s_cnt, s_wcnt);
            uint64_t* k = ki;
            ki = ko;
            ko = k;
            uint32_t* v = vi;
            vi = vo;
            vo = v;
            __threadfence_block();
            __syncthreads();
        }
        for (int e = t; e < m; e += THREADS) {
            const Rec<T> r = recs[vi[e]];
            ko[e] = r.key;
            vo[e] = r.idx;
            put_body<T>(r.x, r.y, r.z, r.m, s0 + e, bodies, bodies32);
        }
        return;
    }
    // sub-buckets: about eight keys each
    int nsub = 16;
    while (nsub < kSub && 8 * nsub < m) nsub *= 2;
    const int ns = min(nsub, m);                     // samples
    // before(k1, e1, k2, e2): place e1's pair comes before place e2's
    auto before = [&](uint64_t k1, int e1, uint64_t k2, int e2) {
        return k1 < k2 || (k1 == k2 && e1 != e2 && recs[e1].idx < recs[e2].idx);
    };
    for (int e = t; e < m; e += THREADS) s_key[e] = recs[e].key;
    if (t < nsub) {
        const int e = (int)((uint32_t)t * (uint32_t)m / (uint32_t)ns);
        s_pk[t] = t < ns ? recs[e].key : ~0ull;
        s_pp[t] = (uint16_t)(t < ns ? e : 0);
        s_rank[t] = t < ns ? 0u : (uint32_t)t;       // fill after the samples
        s_next[t] = 0u;
    }
    __syncthreads();
    // rank the samples, THREADS / nsub threads each against a slice of them
    {
        const int j = t & (nsub - 1), slice = t / nsub, per = max(1, nsub / (THREADS / nsub));
        const int q0 = slice * per, q1 = min(ns, q0 + per);
        if (j < ns && q0 < q1) {
            const uint64_t mk = s_pk[j];
            const int mp = s_pp[j];
            uint32_t lt = 0, le = 0;
#pragma unroll 8
            for (int q = q0; q < q1; ++q) {
                const uint64_t ok = s_pk[q];
                lt += ok < mk ? 1u : 0u;
                le += ok <= mk ? 1u : 0u;
            }
            if (le > lt)                             // itself, and equal keys by index
#pragma unroll 1
                for (int q = q0; q < q1; ++q)
                    if (s_pk[q] == mk) lt += before(mk, s_pp[q], mk, mp) ? 1u : 0u;
            atomicAdd(&s_rank[j], lt);
        }
    }
    __syncthreads();
    if (t < nsub) {
        s_sk[s_rank[t]] = s_pk[t];
        s_sp[s_rank[t]] = s_pp[t];
    }
    __syncthreads();
    // sub-bucket: splitters 1 .. nsub - 1 at or before the pair (the first
    // splitter is left out: it only parts off what lies before the sample)
#pragma unroll 1
    for (int e = t; e < m; e += THREADS) {
        const uint64_t k = s_key[e];
        int p = 0;
#pragma unroll 1
        for (int step = nsub >> 1; step > 0; step >>= 1) {
            const uint64_t sk = s_sk[p + step];
            if (sk < k || (sk == k && !before(k, e, sk, s_sp[p + step]))) p += step;
        }
        s_bin[e] = (uint8_t)p;
        atomicAdd(&s_next[p], 1u);
    }
    __syncthreads();
    if (t < kWave) {
        // two counts per lane of one wave
        const uint32_t c0 = 2 * t < nsub ? s_next[2 * t] : 0u, c1 = 2 * t + 1 < nsub ? s_next[2 * t + 1] : 0u;
        uint32_t x = c0 + c1;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, kWave);
            if (t >= o) x += y;
        }
        s_next[2 * t] = s_start[2 * t] = x - c0 - c1;
        s_next[2 * t + 1] = s_start[2 * t + 1] = x - c1;
        if (t == kWave - 1) s_start[kSub] = x;
    }
    __syncthreads();
#pragma unroll 1
    for (int e = t; e < m; e += THREADS) s_ord[atomicAdd(&s_next[s_bin[e]], 1u)] = (uint16_t)e;
    __syncthreads();
    // each pair's place in its sub-bucket (neighbouring lanes share one, so
    // their places are neighbours too), and its body there
#pragma unroll 1
    for (int p = t; p < m; p += THREADS) {
        const int e = s_ord[p], b = s_bin[e];
        const Rec<T> r = recs[e];
        const uint64_t k = s_key[e];
        const int o0 = (int)s_start[b], o1 = (int)s_start[b + 1];
        uint32_t lt = 0, le = 0;
#pragma unroll 8
        for (int o = o0; o < o1; ++o) {
            const uint64_t ok = s_key[s_ord[o]];
            lt += ok < k ? 1u : 0u;
            le += ok <= k ? 1u : 0u;
        }
        if (le > lt + 1)                             // equal keys by index
#pragma unroll 1
            for (int o = o0; o < o1; ++o)
                if (s_key[s_ord[o]] == k) lt += before(k, s_ord[o], k, e) ? 1u : 0u;
        const int64_t to = s0 + o0 + (int)lt;
        keys_a[to] = r.key;
        idx_a[to] = r.idx;
        put_body<T>(r.x, r.y, r.z, r.m, to, bodies, bodies32);
    }
}

template <typename T, int D>
void split_and_count(const void* pos_, int64_t n, const double* part, int parts, DevParams* prm, const BodySort& a,
                     hipStream_t s) {
    const T* pos = static_cast<const T*>(pos_);
    const BucketShape b = bucket_shape(n);
    const bool fused = b.samples <= kSampleFused;
    uint64_t* skeys = a.keys_b;                      // free until the slow path of k_bucket_sort
    if (!fused)
        hipLaunchKernelGGL((k_sample_keys<T, D>), dim3((unsigned)((b.samples + kRankThreads - 1) / kRankThreads)),
                           dim3(kRankThreads), 0, s, pos, n, part, parts, prm, b.samples, skeys);
    hipLaunchKernelGGL((k_splitters<T, D>), dim3((unsigned)((b.samples + kRankOwn - 1) / kRankOwn)),
                       dim3(kRankThreads), 0, s, pos, n, part, parts, prm, fused ? (const uint64_t*)nullptr : skeys,
                       b.samples, b.samples / b.buckets, b.buckets, a.split_key, a.split_idx);
#define TC_COUNT(TH, PER)                                                                                             \
    hipLaunchKernelGGL((k_bucket_count<T, D, TH, PER>), dim3((unsigned)b.tiles), dim3(TH), 0, s, pos, n,              \
                       (const DevParams*)prm, b.buckets, (const uint64_t*)a.split_key, (const uint32_t*)a.split_idx,  \
                       a.bucket, a.hist)
    if (b.tile == 1024) TC_COUNT(256, 4);
    else if (b.tile == 2048) TC_COUNT(512, 4);
    else if (b.tile == 4096) TC_COUNT(1024, 4);
    else TC_COUNT(1024, 8);
#undef TC_COUNT
}

template <typename T, int D>
void scatter(const void* pos, const void* mass, int64_t n, const DevParams* prm, const BodySort& a, hipStream_t s) {
    const BucketShape b = bucket_shape(n);
    const bool fold = b.tiles <= kFoldTiles;
    if (!fold)
        hipLaunchKernelGGL(k_bucket_scan, dim3((unsigned)(b.buckets / 32)), dim3(1024), 0, s, a.hist, b.tiles,
                           b.buckets, a.total);
#define TC_SCATTER(TH, PER, FOLD)                                                                                    \
    hipLaunchKernelGGL((k_bucket_scatter<T, D, TH, PER, FOLD>), dim3((unsigned)b.tiles), dim3(TH), 0, s,             \
                       static_cast<const T*>(pos), static_cast<const T*>(mass), n, prm, (const uint16_t*)a.bucket,   \
                       b.buckets, (const uint32_t*)a.hist, b.tiles, (const uint32_t*)a.total, a.start,               \
                       static_cast<Rec<T>*>(a.recs))
    if (fold) TC_SCATTER(256, 4, true);              // at most 64 tiles: all of 1024 bodies
    else if (b.tile == 1024) TC_SCATTER(256, 4, false);
    else if (b.tile == 2048) TC_SCATTER(512, 4, false);
    else if (b.tile == 4096) TC_SCATTER(1024, 4, false);
    else TC_SCATTER(1024, 8, false);
#undef TC_SCATTER
}

template <typename T, int D>
void rank_sort(const void* pos, const void* mass, int64_t n, const double* part, int parts, DevParams* prm,
               const BodySort& a, Body* bodies, float4* bodies32, hipStream_t s) {
    hipLaunchKernelGGL((k_rank_sort<T, D>), dim3((unsigned)((n + kRankOwn - 1) / kRankOwn)), dim3(kRankThreads), 0, s,
                       static_cast<const T*>(pos), static_cast<const T*>(mass), (int)n, part, parts, prm, a.keys_a,
                       a.idx_a, bodies, bodies32);
}

template <typename T>
void bucket_sort(int64_t n, const BodySort& a, Body* bodies, float4* bodies32, hipStream_t s) {
    const BucketShape b = bucket_shape(n);
#define TC_BSORT(TH, CAP)                                                                                          \
    hipLaunchKernelGGL((k_bucket_sort<T, TH, CAP>), dim3((unsigned)b.buckets), dim3(TH), 0, s,                     \
                       static_cast<const Rec<T>*>(a.recs), (const uint32_t*)a.start, a.keys_b, a.idx_b, a.keys_a,  \
                       a.idx_a, bodies, bodies32)
    if (n <= 65536) TC_BSORT(256, kBucketCap / 2);   // at most 256 bodies per bucket in the mean
    else TC_BSORT(512, kBucketCap);
#undef TC_BSORT
}

#define TC_BY_TYPE(call)                                      \
    do {                                                      \
        if (f64) {                                            \
            if (dim == 3) { using T = double; constexpr int D = 3; call; } \
            else { using T = double; constexpr int D = 2; call; }          \
        } else {                                              \
            if (dim == 3) { using T = float; constexpr int D = 3; call; }  \
            else { using T = float; constexpr int D = 2; call; }           \
        }                                                     \
    } while (0)

}  // namespace

hipError_t launch_body_keys(const void* pos, int64_t n, int dim, int f64, const double* part, int parts,
                            DevParams* prm, const BodySort& a, hipStream_t s) {
    if (n <= kRankMaxN) return hipSuccess;      // keys and order are one launch there
    TC_BY_TYPE((split_and_count<T, D>(pos, n, part, parts, prm, a, s)));
    return hipGetLastError();
}

hipError_t launch_body_scatter(const void* pos, const void* mass, int64_t n, int dim, int f64, const DevParams* prm,
                               const BodySort& a, hipStream_t s) {
    if (n <= kRankMaxN) return hipSuccess;
    TC_BY_TYPE((scatter<T, D>(pos, mass, n, prm, a, s)));
    return hipGetLastError();
}

hipError_t launch_body_sort(const void* pos, const void* mass, int64_t n, int dim, int f64, const double* part,
                            int parts, DevParams* prm, const BodySort& a, Body* bodies, float4* bodies32,
                            hipStream_t s) {
    if (n <= kRankMaxN) TC_BY_TYPE((rank_sort<T, D>(pos, mass, n, part, parts, prm, a, bodies, bodies32, s)));
    else if (f64) bucket_sort<double>(n, a, bodies, bodies32, s);
    else bucket_sort<float>(n, a, bodies, bodies32, s);
    return hipGetLastError();
}
#undef TC_BY_TYPE

}  // namespace tc
