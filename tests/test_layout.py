"""The carve-up of the workspace: every array that a stage writes lies within
the region it is given, for every number of bodies.  A small host program
(compiled here, linked to the library) asks the library for its regions and
the arrays' places and checks their ends; nothing runs on a GPU."""
import os
import re
import subprocess

import pytest

from paper_1211_2293_amd import build_lib
from paper_1211_2293_amd import treecode as T

PROGRAM = r"""
#include "tc.h"
#include "tc_internal.h"
#include "closure.h"
#include <algorithm>
#include <cstdio>
using namespace tc;

static size_t regions(const Layout& l, size_t* o) {
    const size_t all[] = {@OFFSETS@, l.total};
    std::copy(std::begin(all), std::end(all), o);
    std::sort(o, o + std::size(all));
    return std::size(all);
}

static int bad = 0;
static size_t off[128], noff;

// the array of `bytes` at `begin` ends within the region that it begins in
static void holds(const Layout& l, const char* what, size_t begin, size_t bytes) {
    const size_t end = *std::upper_bound(off, off + noff, begin);
    if (begin + bytes > end && bad++ < 20)
        printf("n=%lld dim=%d leaf_cap=%d: %s needs %zu bytes, its region has %zu\n", (long long)l.n, l.dim, l.leaf_cap, what,
               bytes, end - begin);
}

static void check(int64_t n, int dim, int leaf_cap) {
    const Layout l = make_layout(n, dim, leaf_cap);
    noff = regions(l, off);
    auto ws = reinterpret_cast<uint8_t*>(uintptr_t(1) << 40);
    auto at = [&](const void* p) { return (size_t)(static_cast<const uint8_t*>(p) - ws); };
    const size_t N = (size_t)n, C = (size_t)l.cmax, G = (size_t)l.gmax;
    if (n < kBucketMaxN) {
        const BodySort a = body_sort_arrays(l, ws);
        holds(l, "sorted keys", at(a.keys_a), 8 * N);
        holds(l, "permutation", at(a.idx_a), 4 * N);
        if (n > kRankMaxN) {
            const BucketShape b = bucket_shape(n);
            const size_t B = b.buckets;
            holds(l, "sample keys", at(a.keys_b), 8 * std::max<size_t>(N, b.samples));
            holds(l, "indices on their way", at(a.idx_b), 4 * N);
            holds(l, "bucket numbers", at(a.bucket), 2 * N);
            holds(l, "counts per tile and bucket", at(a.hist), 4 * B * b.tiles);
            holds(l, "records", at(a.recs), 48 * N);
            holds(l, "splitters and starts", at(a.split_key), 8 * B + 4 * B + 4 * B + 4 * (B + 1));
            if (at(a.start) + 4 * (B + 1) > at(a.split_key) + 20 * B + 4 && bad++ < 20) printf("starts at n=%lld\n", (long long)n);
        }
    }
    // the radix sorts: counts per digit and tile (of the bodies and of the cells by level)
    holds(l, "radix counts", l.off_hist, 4 * 256 * (size_t)sort_tiles(n));
    holds(l, "level counts", l.off_lvl_hist, 4 * 256 * ((C + 1023) / 1024));
    holds(l, "packed input", l.off_recs, 32 * N);
    // boxes, then the counters of the upper cells in their place
    holds(l, "partial boxes", l.off_bbox_part, 56 * (size_t)bbox_parts(n));
    holds(l, "upper counters", l.off_bbox_part, 4 * kLevels * BigList::kStride);
    const size_t cap = C / (subtree_cells(l.cmax) + 1);
    holds(l, "upper cells", l.off_big, 4 * kLevels * cap);
    // scratch of the mid-size trees
    holds(l, "cells per body tile", l.off_idx_b, 4 * (N / 256 + 1));
    holds(l, "cells per level and tile", l.off_lvl_hist, 4 * kLevels * (C / 1024 + 1));
    holds(l, "groups per tile", l.off_goff, 4 * (C / 1024 + 1));
    // the schedule's places, costs and keys
    holds(l, "group order", l.off_gorder, 10 * G);
    // training pairs: keys, offsets, counters
    const size_t keys = std::min<size_t>(kResidKeys, C);
    holds(l, "pairs per key", l.off_gper, 4 * keys);
    holds(l, "pairs' offsets", l.off_goff, 4 * (keys + 1));
    holds(l, "pairs' partial sums", l.off_gscan_part, 4 * ((keys + kScanTile - 1) / kScanTile));
    holds(l, "pair counters", l.off_rcount, 4 * (1 + 2 * 16) * 32);
}

int main() {
    long cases = 0;
    auto sweep = [&](int64_t lo, int64_t hi, int64_t step, int dim, int leaf_cap) {
        for (int64_t n = lo; n < hi; n += step, ++cases) check(n, dim, leaf_cap);
    };
    sweep(1, kBucketMaxN + 3, 1, 3, 16);                       // every size that the body sort takes
    for (int dim = 2; dim <= 3; ++dim)
        for (int leaf_cap : {1, 2, 16, 256}) {
            sweep(1, 9000, 1, dim, leaf_cap);
            sweep(9001, kBucketMaxN + 997, 997, dim, leaf_cap);
            sweep(3000000, 8000000, 499979, dim, leaf_cap);
        }
    printf("%ld cases, %d too small\n", cases, bad);
    return bad != 0;
}
"""


def test_every_region_holds_its_arrays(tmp_path):
    T.lib()                                # built if nothing is
    with open(os.path.join(build_lib.CSRC, "tc_internal.h")) as f:
        layout = re.search(r"struct Layout \{(.*?)\n\};", f.read(), re.S).group(1)
    names = sorted(set(re.findall(r"\boff_\w+", layout)))
    assert len(names) > 40
    src = tmp_path / "layout.hip"
    src.write_text(PROGRAM.replace("@OFFSETS@", ", ".join("l." + n for n in names)))
    exe = tmp_path / "layout"
    pkg = os.path.dirname(build_lib.LIB)
    subprocess.run([build_lib.HIPCC, *build_lib.CFLAGS, str(src), "-o", str(exe), "-L", pkg, "-l:libtc.so",
                    f"-Wl,-rpath,{pkg}"], check=True, capture_output=True, text=True, timeout=300)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(p.stdout)
    assert p.returncode == 0, p.stdout + p.stderr
