// Internal declarations shared by the HIP translation units of libtc.
// Not part of the public ABI (include/tc.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace tc {

constexpr int kWave = 64;           // CDNA wavefront width
constexpr int kGroup = 64;          // bodies per walk group = one wave
constexpr int kMaxLeafCap = 256;    // the largest leaf_cap (TC_MAX_LEAF_CAP)
// Radix-sort tiles: 256 threads x sort_per(n) keys.  One block per tile
// and few blocks leave the passes latency-bound, so smaller sorts use
// smaller tiles (measured per pass: 1M keys 16.0 us with 4096-key tiles,
// 16.6 with 2048, 18.6 with 1024; 262k keys 14.2 us with 4096, 9.4 with
// 2048, 7.3 with 1024): the largest tile that still gives 256 tiles.
inline int sort_per(int64_t n) { return n >= (int64_t)256 * 4096 ? 16 : n >= (int64_t)256 * 2048 ? 8 : 4; }
inline int64_t sort_tiles(int64_t n) { return (n + 256 * sort_per(n) - 1) / (256 * sort_per(n)); }
// Tiles a histogram buffer must hold for any sort of at most n keys.
inline int64_t sort_tiles_max(int64_t n) { return (n + 1023) / 1024; }
constexpr int kScanTile = 4096;     // elements per scan tile
constexpr int kDiagBlocks = 512;    // fixed partial count of the FP64 diagnostics
constexpr int kCluster = 1024;      // walk groups never straddle a cell of <= kCluster bodies
constexpr int kXcd = 8;             // XCDs per MI355X: one work queue each
constexpr int kQueueStride = 64;    // work-queue counters 256 B apart (own cache lines)

// Status bits raised by kernels into the workspace's status word.
constexpr uint32_t kFlagNonFinite = 1u;
constexpr uint32_t kFlagOverflow = 2u;   // cell bound exceeded (never expected)
constexpr uint32_t kFlagBadIndex = 4u;   // an index argument outside its array

inline int levels_for(int dim) { return dim == 3 ? 21 : 31; }

// A body in key order: FP64 position and mass (z = 0 in 2D).
struct __align__(32) Body {
    double x, y, z, m;
};

// Topology of one cell (pre-order index k).
struct __align__(16) Cell {
    uint64_t prefix;   // key prefix: the top level*dim bits of its bodies' keys
    int32_t begin;     // first sorted body
    int32_t count;     // number of bodies
    int32_t skip;      // pre-order index just past the subtree
    int32_t parent;    // -1 for the root
    int32_t level;
    int32_t leaf_nch;  // bit 31: leaf; low bits: number of children
};

// FP64 moments of one cell: total mass, mass-weighted position sum, centre
// of mass and traceless quadrupole (xx, yy, zz, xy, xz, yz).
struct __align__(16) Moments {
    double M;
    double S[3];
    double com[3];
    double Q[6];
    double pad;
};

// What the walk reads per cell, in level order (breadth-first: all cells of
// level 0, then level 1, ...; within a level in pre-order), so that the
// children of every cell are contiguous.  48 bytes, one lane per cell.
//   a = leaf ? first sorted body : level-order index of the first child
//   b = leaf ? (body count | 0x80000000) : number of children
struct __align__(16) WalkCell {
    double cx, cy, cz;   // centre of mass (FP64)
    double rcrit2;       // squared opening radius for the current theta
    float m;             // total mass, FP32
    int32_t a;
    int32_t b;
    int32_t pad;
};

// Device-side scalars computed by the kernels.
struct DevParams {
    double lo[3];        // root cube corner
    double size;         // root cube side (a power of two)
    double scale;        // 2^L / size
    uint32_t ncells;
    uint32_t status;     // kFlag* bits, sticky until the next build
    uint32_t ngroups;    // walk groups of the current tree
    uint32_t pad;
};

// The moments pass does the maximal subtrees of at most subtree_cells(cmax)
// cells within a block and the cells above them level by level: smaller
// subtrees leave more blocks per CU, larger ones fewer cells above (which one
// block does, except in the largest trees).  Measured (both kernels, 128 / 256
// cells): 36 / 38 us at 50,000 bodies, 38 / 40 at 100,000, 42 / 42 at 200,000, 45 / 43
// at 230,000 (2^19 slots are 235,000 bodies in leaves of 16), 47 / 50 at 300,000, 61 /
// 56 at 500,000, 101 / 88 at 1M, 146 / 142 at 1.8M; 135 / 140 at 2M (past 2^22 slots,
// where the levels above get launches of their own), 169 / 183 at 3M, 726 / 790 at
// 16.7M; 2D 33 / 31 at 300,000, 81 / 75 at 1.4M, 117 / 123 at 3M.
inline int subtree_cells(int64_t cmax) {
    return cmax < (int64_t)1 << 19 || cmax >= (int64_t)1 << 22 ? 128 : 256;
}
constexpr int kSubtreeMin = 128;
// The cells above, one list per level (in any order; at most cap = cmax /
// (sub + 1) per level, whose subtrees are disjoint).
constexpr int kLevels = 32;                      // levels 0..21 in 3D, 0..31 in 2D
struct BigList {
    static constexpr int kStride = 32;           // counters 128 B apart (own cache lines)
    static constexpr int kWide = 1;              // beside the first: the moments' window of levels
    uint32_t* count;                             // [kLevels * kStride]
    uint32_t* cell;                              // [kLevels][cap]: pre-order indices
    uint32_t cap;
    int sub;                                     // subtree_cells
};

// Carve-up of the caller's workspace.
struct Layout {
    int64_t n;
    int dim, leaf_cap;
    int64_t cmax;        // cell bound
    int64_t groups;      // ceil(n / 64)
    int64_t sort_tiles;
    int64_t scan_tiles;
    size_t off_params, off_keys_a, off_keys_b, off_idx_a, off_idx_b, off_bodies, off_range,
        off_nper, off_cstart, off_scan_part, off_hist, off_digit_tot, off_cells, off_mom,
        off_walk, off_recs, off_big, off_bodies32, off_acc, off_pot, off_m2p, off_p2p, off_bbox_part, off_diag_part,
        off_diag_out, off_lvl_idx_b, off_pre2bfs,
        off_lvl_hist, off_gper, off_goff, off_gscan_part, off_gbeg, off_gcnt, off_queue, off_gorder, off_bcost, off_lvl_off, off_inv_perm, off_rcount, off_roffs,
        off_rscan_part, off_mlp, off_rcp2, off_nlearn, off_nfall, off_pb_cnt, off_pb_off, off_pb_part, off_walkq, off_split, off_tests, total;
    int64_t lvl_tiles;   // radix tiles over cmax cells (level sort)
    int64_t gmax;        // bound on walk groups
    int64_t cscan_tiles; // scan tiles over cmax cells
};

Layout make_layout(int64_t n, int dim, int leaf_cap);

// ---- launchers (all enqueue on `s`, return hipSuccess or the launch error)
// build.hip
// Partial boxes of the input, bbox_parts(n) of 7 doubles.  With `packed` it also
// packs the input into (x, y, z, m) records (float4, or double4 for FP64
// input; n of them) for launch_gather and reduces the boxes to the root cube;
// without, the kernels of bodysort.hip do that.
int bbox_parts(int64_t n);
// A step's half kick and drift, folded into the pass over the bodies' box.
struct KickDrift {
    void* vel;
    const float* acc;
    double dt;
};
// pos is written only with kick.
hipError_t launch_bbox(void* pos, const void* mass, int64_t n, int dim, int f64, double* part, void* packed,
                       const KickDrift* kick, DevParams* prm, hipStream_t s);
hipError_t launch_keys(const void* pos, int64_t n, int dim, int f64, const DevParams* prm,
                       uint64_t* keys, uint32_t* idx, hipStream_t s);
// LSD radix sort (stable) of the low key_bits bits; idx_a / idx_b may both be
// null for keys without a payload.
// hist holds 256 x sort_tiles_max(n) counts.
hipError_t launch_sort(uint64_t* keys_a, uint32_t* idx_a, uint64_t* keys_b, uint32_t* idx_b,
                       int64_t n, int key_bits, uint32_t* hist, uint32_t* digit_tot, hipStream_t s);
hipError_t launch_gather(const void* packed, const uint32_t* perm, int64_t n, int f64, Body* bodies,
                         float4* bodies32, hipStream_t s);
// bodysort.hip: keys, order and gather of fewer than kBucketMaxN bodies, from
// the input and the partial boxes of launch_bbox (whose root cube it stores
// in prm).  Three parts in this order; small systems do all in the last.
// keys_a and idx_a receive the sorted keys and the permutation.
constexpr int64_t kRankMaxN = 8192;
constexpr int64_t kBucketMaxN = (int64_t)1 << 21;
// Buckets, samples and tiles for n bodies: about 256 bodies per bucket while
// few buckets leave CUs idle, at most 1024 (a quarter of what a block can
// sort in LDS); the tiles grow with the buckets, so a tile's counts are a
// quarter of a full tile's bodies (the last tile, full or not, has as many).
// Eight samples per bucket bound its size by four times the mean but for
// about 1e-7 of the buckets; four do for smaller means.
struct BucketShape {
    int buckets, samples, tile, tiles;
};
inline BucketShape bucket_shape(int64_t n) {
    BucketShape b;
    if (n <= 65536) {
        b.buckets = 32;
        while (256 * (int64_t)b.buckets < n) b.buckets *= 2;
        b.tile = 1024;
    } else {
        b.buckets = 256;
        while (1024 * (int64_t)b.buckets < n) b.buckets *= 2;
        b.tile = 4 * b.buckets;
    }
    b.samples = b.buckets * (n > 512 * (int64_t)b.buckets ? 8 : 4);
    b.tiles = (int)((n + b.tile - 1) / b.tile);
    return b;
}
struct BodySort {
    uint64_t *keys_a, *keys_b;   // [n]
    uint32_t *idx_a, *idx_b;     // [n]
    uint16_t* bucket;            // [n]
    uint32_t* hist;              // [tiles][buckets]
    void* recs;                  // 48 n bytes
    uint64_t* split_key;         // [buckets]
    uint32_t *split_idx, *total, *start;   // [buckets], [buckets], [buckets + 1]
};
// Its arrays in the workspace ws (api.hip).
BodySort body_sort_arrays(const Layout& l, uint8_t* ws);
hipError_t launch_body_keys(const void* pos, int64_t n, int dim, int f64, const double* part, int parts,
                            DevParams* prm, const BodySort& a, hipStream_t s);
hipError_t launch_body_scatter(const void* pos, const void* mass, int64_t n, int dim, int f64, const DevParams* prm,
                               const BodySort& a, hipStream_t s);
hipError_t launch_body_sort(const void* pos, const void* mass, int64_t n, int dim, int f64, const double* part,
                            int parts, DevParams* prm, const BodySort& a, Body* bodies, float4* bodies32,
                            hipStream_t s);
// Mid-size trees: the same topology, level order and walk groups as
// launch_topology, launch_level_order and launch_groups, with their scans
// folded in.  Each block of 1024 cells reads the level counts of all of them,
// so this is for at most a few hundred such tiles, by the host's estimate of
// the cells.
inline bool fused_tree(int64_t n, int64_t cells_est) { return n < kBucketMaxN && cells_est <= (int64_t)1 << 19; }
struct TreeScratch {
    uint32_t* tile_tot;          // [n / 256 + 1]
    uint32_t* hist;              // [cmax / 1024 + 1][kLevels]
    uint32_t* gtile;             // [cmax / 1024 + 1]
};
hipError_t launch_tree_cells(const uint64_t* keys, int64_t n, int dim, int leaf_cap, uint32_t* range, uint32_t* nper,
                             uint32_t* cstart, Cell* cells, int64_t cmax, DevParams* prm, const BigList& big,
                             const TreeScratch& a, hipStream_t s);
hipError_t launch_tree_link(Cell* cells, int64_t cmax, int dim, const DevParams* prm, const BigList& big,
                            uint32_t* bfs2pre, uint32_t* pre2bfs, uint32_t* lvl_off, uint32_t* gper,
                            const TreeScratch& a, hipStream_t s);
hipError_t launch_tree_groups(const Cell* cells, int64_t cmax, const uint32_t* gper, int32_t* gbeg, int32_t* gcnt,
                              int64_t gmax, DevParams* prm, const TreeScratch& a, hipStream_t s);
hipError_t launch_topology(const uint64_t* keys, int64_t n, int dim, int leaf_cap,
                           uint32_t* range, uint32_t* nper, uint32_t* cstart,
                           uint32_t* scan_part, int64_t scan_tiles, Cell* cells,
                           int64_t cmax, DevParams* prm, const BigList& big, hipStream_t s);
// Level order (one radix pass by level over the live cells): bfs2pre and
// pre2bfs, and lvl_off, where each level starts (levels 0..L and the end).
// cells_est, an estimate of the live cells (any value works), sets the tile.
hipError_t launch_level_order(const Cell* cells, int64_t cmax, int64_t cells_est, int dim, const DevParams* prm, uint32_t* bfs2pre,
                              uint32_t* hist, uint32_t* digit_tot, uint32_t* pre2bfs, uint32_t* lvl_off,
                              hipStream_t s);
hipError_t launch_groups(const Cell* cells, int64_t cmax, uint32_t* gper, uint32_t* goff, uint32_t* scan_part,
                         int64_t scan_tiles, int32_t* gbeg, int32_t* gcnt, int64_t gmax, DevParams* prm,
                         hipStream_t s);
hipError_t launch_moments(const Cell* cells, const Body* bodies, int dim, int64_t cmax, const uint32_t* bfs2pre,
                          const uint32_t* pre2bfs, const BigList& big, const DevParams* prm, Moments* mom,
                          WalkCell* walk, hipStream_t s);
hipError_t launch_mac(const Cell* cells, const Moments* mom, int dim, double theta, int64_t cmax,
                      const uint32_t* pre2bfs, WalkCell* walk, double* rc_out, const DevParams* prm,
                      hipStream_t s);
hipError_t launch_export(const Cell* cells, const Moments* mom, int dim, int64_t cmax,
                         const DevParams* prm, int32_t* level, uint64_t* prefix, int32_t* begin,
                         int32_t* count, int32_t* parent, int32_t* skip, int32_t* nch,
                         int32_t* leaf, double* M, double* com, double* Q, hipStream_t s);
// force.hip
// order: room for 2 gmax uint32 (places, costs) and gmax uint16 keys; bcost:
// n uint32 per-body list lengths, written for the next call's schedule.
// Where the force kernels put their results: the copies that the next step and
// the diagnostics read and, where given, the caller's arrays.
struct ForceOut {
    float *acc, *pot, *user_acc, *user_pot;
    __device__ __forceinline__ void put_acc(int64_t at, float v) const {
        acc[at] = v;
        if (user_acc) user_acc[at] = v;
    }
    __device__ __forceinline__ void put_pot(int64_t at, float v) const {
        pot[at] = v;
        if (user_pot) user_pot[at] = v;
    }
    // body o's whole result, its components side by side in each array
    template <int D>
    __device__ __forceinline__ void put(int64_t o, float x, float y, float z, float p) const {
        put_vec<D>(acc + o * D, x, y, z);
        pot[o] = p;
        if (user_acc) put_vec<D>(user_acc + o * D, x, y, z);
        if (user_pot) user_pot[o] = p;
    }
    template <int D>
    static __device__ __forceinline__ void put_vec(float* a, float x, float y, float z) {
        a[0] = x;
        a[1] = y;
        if (D == 3) a[2] = z;
    }
};
// Up to direct_out_max bodies the kernels store into the caller's arrays too;
// beyond, the arrays are copied: bodies lie in the caller's order, so the
// stores go to scattered lines, and a second set of these costs more than two
// copies once the sets outgrow the caches, the sooner the less else the kernel
// does.  Measured (tc_forces, stores / copies, us): 3D 10,000 bodies 57 / 62,
// 1,300,000 2,133 / 2,118, 2,000,000 3,262 / 3,234 and at theta 1 1,214 / 1,185,
// 4,000,000 (theta 1) 1,917 / 1,892; 2D, theta 0.5 and 0.9, 400,000 188 / 192 and
// 135 / 138, 700,000 289 / 293 and 231 / 231, 1,000,000 420 / 430 and 327 / 316,
// 2,000,000 758 / 743 and 591 / 570.
inline int64_t direct_out_max(int dim) { return dim == 3 ? 3 << 19 : 3 << 18; }
hipError_t launch_walk_force(const WalkCell* walk, const float4* walkq, const Body* bodies, const float4* bodies32,
                             const uint32_t* perm,
                             const int32_t* gbeg, const int32_t* gcnt, int64_t gmax, uint32_t* order,
                             uint32_t* queue, uint32_t* bcost, int64_t n, int dim, int leaf_cap, float G, float eps2,
                             const DevParams* prm, const ForceOut& out, int64_t* m2p,
                             int64_t* p2p, int64_t* tests, bool plain, bool share,
                             double theta, hipStream_t s);
hipError_t launch_scan_u32(const uint32_t* in, int64_t n, uint32_t* out, uint32_t* part, int64_t tiles,
                           hipStream_t s);
// closure.hip
struct MlpState;
hipError_t launch_direct64(const Body* bodies, const uint32_t* inv_perm, int64_t n, const int32_t* targets, int nt,
                           double eps2, double G, DevParams* prm, double* acc, double* pot, hipStream_t s);
// Split walks pay off for small n only (measured on 3D Plummer spheres:
// 1.6x faster force evaluations at 2,000 bodies, 1.14x at 10,000, 0.64x at
// 16,384; on 2D disks 1.25x at 16,384, 0.90x at 32,768).  The shared walks
// below are faster still, so split walks are used only when asked for
// (tc_set_split(ctx, 2)), for n at most split_max_n(dim); the workspace holds
// their partial sums.
constexpr int64_t kSplitMaxN3 = 12288;
constexpr int64_t kSplitMaxN2 = 24576;
inline int64_t split_max_n(int dim) { return dim == 3 ? kSplitMaxN3 : kSplitMaxN2; }
// Up to coop_max_n bodies, one block of waves shares each group's walk and
// list (k_walk_force_coop); beyond, one wave per group.  Shared walks pay by
// evening out the lists, the less the shorter these are, so in 3D the line
// falls as theta rises, and it is lower with quadrupoles, whose sums weigh
// more.  Measured (tc_forces in us, one wave / shared):
//   3D Plummer, theta 0.5: 347 / 57 at 10,000 bodies, 544 / 479 at 262,144,
//     716 / 686 at 400,000, 880 / 879 at 524,288; theta 0.7: 360 / 340 at
//     330,000, 388 / 405 at 400,000; theta 1: 205 / 208 at 262,144, 341 / 380 at
//     524,288;
//   3D cube, theta 0.5: 592 / 593 at 524,288; theta 0.7: 236 / 235 at 330,000,
//     337 / 369 at 524,288; theta 1: 128 / 124 at 200,000, 246 / 283 at 524,288;
//   quadrupoles, Plummer and cube, theta 0.3: 4,993 / 4,383 and 2,263 / 2,277 at
//     524,288; theta 0.5: 1,186 / 1,169 and 646 / 668 at 400,000; theta 0.7: 476 /
//     451 and 236 / 246 at 262,144; theta 1: 270 / 252 and 170 / 157 at 200,000,
//     363 / 386 and 230 / 238 at 330,000;
//   2D disk: 107 / 85 at 163,840 (theta 0.5) and 79 / 68 (theta 1), 115 / 143
//     at 262,144.
// tc_set_split(ctx, 0) turns it off; tc_set_split(ctx, 2) uses the split walks
// (above) for n <= split_max_n(dim) instead.
constexpr int64_t kCoopMaxN2 = 163840;
inline int64_t coop_max_n(int dim, double theta, bool quad) {
    if (dim != 3) return kCoopMaxN2;
    const double line = quad ? 196608 : 262144;          // theta n up to which sharing pays
    return theta * 524288 <= line ? 524288 : (int64_t)(line / theta);
}
// How a block shares a group: its waves, the tasks (of 64 / parts bodies) a
// group is cut into, and whether the longest walks are sent first
// (k_group_order).  More waves shorten one group's walk and sums, where the
// chip has blocks to spare; fewer let more blocks share a CU, whose walks
// and sums then overlap.  Measured (force evaluation in us, 3D Plummer):
// 10,000 bodies, 8 waves x 2 parts 61, 8 x 1 78, 8 x 4 83, 4 x 1 113, 16 x
// 1 77; 20,000: 8 x 1 86, 4 x 2 100, 8 x 2 107, 4 x 1 108; 35,000: 8 x 1
// 108, 4 x 1 122; 50,000: 4 x 1 149, 8 x 1 160, 2 x 1 208; 100,000: 219,
// 267, 276.  2D disk (theta 0.5): 20,000: 8 waves 34, 4 waves 38; 40,000: 4 waves
// 40, 8 waves 48; 100,000: 2 waves 66, 4 waves 66.  There four waves hold out
// longer at a small theta, whose lists are long (theta 0.3 / 0.7 / 1, 4 and 2
// waves: 70,000 bodies 67 43 39 and 81 49 46; 90,000 82 53 51 and 98 52 45;
// 140,000 113 81 79 and 111 57 51).  While about every task has a block of its
// own (12,288 bodies of two tasks a group, 30,000 of one in 2D, where the walks
// differ least) the order is skipped: 4,096 bodies in 3D 31 -> 24 us, 14,000 in
// 2D 32 -> 23, 30,000 37 -> 29.
struct CoopShape {
    int waves, parts;
    bool ordered;
};
inline CoopShape coop_shape(int64_t n, int dim, double theta) {
    if (dim == 3) return n <= 12288 ? CoopShape{8, 2, false} : CoopShape{n <= 40000 ? 8 : 4, 1, true};
    if (n <= 30000) return {8, 1, false};
    const double k = (double)n / 100000;                 // 4 waves up to 100,000 sqrt(0.5 / theta) bodies
    return {k * k * theta <= 0.5 ? 4 : 2, 1, true};
}
hipError_t launch_walk_force_split(const WalkCell* walk, const float4* walkq, const Body* bodies,
                                   const float4* bodies32, const uint32_t* perm, const int32_t* gbeg,
                                   const int32_t* gcnt, int64_t gmax, int64_t n, int dim, int leaf_cap, float G,
                                   float eps2, const DevParams* prm, float4* part, const ForceOut& out,
                                   int64_t* m2p, int64_t* p2p, int64_t* tests, bool plain, hipStream_t s);
hipError_t launch_quad_pack(const Moments* mom, const uint32_t* pre2bfs, const DevParams* prm, int64_t cmax,
                            float4* walkq, hipStream_t s);
// perbody.hip
hipError_t launch_pb_count(const WalkCell* walk, const Body* bodies, int64_t n, int dim, uint32_t* counts,
                           uint64_t* offs, uint64_t* part, hipStream_t s);
hipError_t launch_pb_write_sum(const WalkCell* walk, const Body* bodies, const uint32_t* perm, int64_t n, int dim,
                               const uint64_t* offs, uint32_t* lists, int64_t cap, int64_t cbound, float G,
                               float eps2, float* acc, float* pot, hipStream_t s);
hipError_t launch_inverse_perm(const uint32_t* perm, int64_t n, uint32_t* inv, hipStream_t s);
hipError_t launch_resid_count(const WalkCell* walk, const Body* bodies, const uint32_t* bfs2pre,
                              const uint32_t* inv_perm, DevParams* prm, int64_t n, const int32_t* targets, int nt,
                              uint32_t* counts, hipStream_t s);
// Keys of the order by cell: the first cells in level order, which hold nearly
// all the large ones, have one key each.  Fewer keys cost fewer atomics in the
// list pass but lose the pairs side by side (4,096 targets, 1,000,001 bodies: 2.76
// ms with 2,048 keys, 2.21 with 4,096, 1.98 with 16,384).
constexpr int64_t kResidKeys = 16384;
constexpr uint32_t kResidColdKeys = 256;
// Up to kResidSmall bodies the pairs are one launch instead of seven (us for a
// call of 1, 128 and all targets, theta 0.9, seven / one: 100 bodies 94, 99, 99 /
// 53, 60, 60; 800: 97, 108, 144 / 62, 113, 106; 1,200: 97, 109, 173 / 66, 110, 125;
// 2,000: 99, 117, 273 / 80, 181, 248).
constexpr int64_t kResidSmall = 1024;
hipError_t launch_resid_pairs(const WalkCell* walk, const Body* bodies, const float4* bodies32, const Cell* cells, const Moments* mom,
                              const uint32_t* bfs2pre, const uint32_t* pre2bfs, const uint32_t* inv_perm,
                              DevParams* prm, int64_t n, int64_t cmax, const int32_t* targets, int nt, double eps2,
                              const uint32_t* offs, int64_t cap, uint32_t* key_count, uint32_t* key_off,
                              uint32_t* key_part, uint32_t* ctr, float* feat, float* y, int32_t* cell_out,
                              hipStream_t s);
hipError_t launch_mlp_load(MlpState* st, const float* params, hipStream_t s);
hipError_t launch_mlp_get(const MlpState* st, float* params, hipStream_t s);
hipError_t launch_mlp_forward(const MlpState* st, const float* feat, int64_t nrows, const int32_t* idx, int64_t nb,
                              float* yhat, uint32_t* status, hipStream_t s);
hipError_t launch_mlp_step(MlpState* st, const float* feat, const float* y, int64_t nrows, const int32_t* idx,
                           int64_t nb, float lr, int step, float* grad_out, uint32_t* status, hipStream_t s);
// learned.hip
hipError_t launch_walk_force_learned(const WalkCell* walk, const double* rcp2, const Body* bodies,
                                     const float4* bodies32, const Cell* cells, const Moments* mom,
                                     const uint32_t* bfs2pre, const uint32_t* perm, const int32_t* gbeg,
                                     const int32_t* gcnt, int64_t gmax, uint32_t* queue, const MlpState* st,
                                     int leaf_cap, float G, float eps2, float tau, int64_t n,
                                     const DevParams* prm, float* acc, float* pot, int64_t* m2p, int64_t* p2p,
                                     int64_t* learned, int64_t* fallback, hipStream_t s);
// fmm.hip
// Geometric centre of a cell, the centre of its local expansion.
struct __align__(16) FmmGeo {
    double z[3];
    double pad[5];
};
// What the traversal reads of a cell, in level order: centre, centre of
// mass, the radii bounding its bodies about the two (rhoA, rhoB), its first child (level order; children are
// contiguous there), child count with bit 31 set for a leaf, and level.
constexpr int kFmmMaxWaves = 8192;      // waves per traversal launch: what the chip holds at once
// Counters of the traversal: [1], [2] M2L and P2P pairs so far; from kFmmSizes
// on a ring of level sizes; of the leaf tasks: [3] tasks << 32 | long ones,
// [0] partial slots.
constexpr int kFmmCounters = 32, kFmmSizes = 4, kFmmRing = kFmmCounters - kFmmSizes;
struct __align__(16) DttCell {
    double z[3];
    double com[3];
    double rhoA, rhoB;
    int32_t child, nch_leaf, level, pre;   // pre: the cell's pre-order index
};
hipError_t launch_fmm_geo(const Cell* cells, const Moments* mom, const Body* bodies, const WalkCell* walk,
                          const uint32_t* pre2bfs, const DevParams* prm, int64_t cmax, FmmGeo* geo, DttCell* dc,
                          hipStream_t s);
hipError_t launch_fmm_radii(const uint32_t* lvl_off, int level, int64_t count, DttCell* dc, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, int64_t n, hipStream_t s);
hipError_t launch_fmm_dtt_root(unsigned long long* ctr, uint64_t* fin, hipStream_t s);
hipError_t launch_fmm_dtt(const DttCell* dc, const uint32_t* bfs2pre, double theta, uint64_t* fin, int64_t bound,
                          const unsigned long long* size, unsigned long long* next, uint64_t* fout, int64_t capf,
                          uint64_t* m2l, int64_t capm, uint64_t* p2p, int64_t capp, unsigned long long* ctr,
                          uint32_t* bt, unsigned long long* base, hipStream_t s);
hipError_t launch_fmm_offsets(const uint64_t* keys, int64_t n, int64_t C, uint32_t* off, hipStream_t s);
hipError_t launch_fmm_m2l(const Moments* mom, const FmmGeo* geo, const DevParams* prm, int64_t cmax,
                          const uint64_t* keys, const uint32_t* off, double eps2, double* lam,
                          hipStream_t s);
hipError_t launch_fmm_l2l(const Cell* cells, const FmmGeo* geo, const uint32_t* bfs2pre, const uint32_t* lvl_off,
                          int level, int64_t count, double* lam, hipStream_t s);
hipError_t launch_fmm_tasks(const Cell* cells, const uint32_t* poff, const DevParams* prm, int64_t cmax,
                            uint32_t* ntask, uint32_t* nslot, unsigned long long* ctr, hipStream_t s);
hipError_t launch_fmm_tasks_fill(const uint32_t* toff, const uint32_t* poff, const DevParams* prm, int64_t cmax,
                                 uint32_t* task, uint32_t* longs, unsigned long long* ctr, hipStream_t s);
hipError_t launch_fmm_leaf(const Cell* cells, const Body* bodies, const float4* bodies32, const uint32_t* perm,
                           const FmmGeo* geo, const double* lam, const uint64_t* pkeys, const uint32_t* poff,
                           const uint32_t* task, const uint32_t* toff, const uint32_t* soff, int64_t ntasks,
                           const uint32_t* longs, int64_t nlong,
                           double* part, const DevParams* prm, int64_t cmax, float G, float eps2, float* acc,
                           float* pot, hipStream_t s);
hipError_t launch_fmm_unpack(const uint64_t* keys, int64_t n, int32_t* out, hipStream_t s);
// step.hip
hipError_t launch_kick_drift(void* pos, void* vel, const float* acc, int64_t n, int dim, int f64,
                             double dt, hipStream_t s);
hipError_t launch_kick(void* vel, const float* acc, int64_t n, int dim, int f64, double dt,
                       hipStream_t s);
hipError_t launch_diag(const void* mass, const void* vel, const float* acc, const float* pot,
                       int64_t n, int dim, int f64, double* part, double* out, hipStream_t s);

// Grid size for grid-stride loops over `work` items with 256-thread blocks.
inline unsigned grid_for(int64_t work, int64_t cap = 16384) {
    int64_t b = (work + 255) / 256;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

}  // namespace tc
