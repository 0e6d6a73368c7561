"""GPU tree construction vs the oracle, bit for bit: root cube, Morton keys,
stable sort order, cell topology in pre-order, FP64 moments (§3.1)."""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import assert_tree_equal, gpu_tree

pytestmark = pytest.mark.gpu


def _grid_faces(n=512):
    # bodies exactly on subdivision planes (dyadic coordinates)
    rng = np.random.default_rng(40)
    return (rng.integers(0, 9, (n, 3)) / 8.0).astype(np.float32)


def _two_clumps(n=3000):
    rng = np.random.default_rng(41)
    a = rng.normal(0.2, 1e-4, (n // 2, 3))
    b = rng.normal(0.8, 1e-5, (n - n // 2, 3))
    return np.concatenate([a, b]).astype(np.float32)


CASES = {
    "uniform-cube-4096-f64": lambda: (workloads.uniform_cube(4096).pos, np.full(4096, 1 / 4096), 8),
    "uniform-5000-f32": lambda: (np.random.default_rng(42).uniform(-1, 3, (5000, 3)).astype(np.float32),
                                 np.random.default_rng(43).uniform(0.5, 2, 5000).astype(np.float32), 16),
    "plummer-20000": lambda: (workloads.plummer_sphere(20000, seed=44).pos,
                              workloads.plummer_sphere(20000, seed=44).mass, 16),
    "disk2d-9000": lambda: (workloads.gaussian_disk(9000, seed=45).pos,
                            workloads.gaussian_disk(9000, seed=45).mass, 16),
    "disk2d-lc1": lambda: (workloads.gaussian_disk(700, seed=46).pos,
                           workloads.gaussian_disk(700, seed=46).mass, 1),
    "clustered-20000": lambda: (workloads.clustered(20000, seed=47).pos,
                                workloads.clustered(20000, seed=47).mass, 16),
    "faces-512": lambda: (_grid_faces(), np.ones(512, np.float32), 4),
    "two-clumps": lambda: (_two_clumps(), np.ones(3000, np.float32), 8),
    "coincident-100": lambda: (np.full((100, 3), 0.5, np.float32), np.ones(100, np.float32), 8),
    "one-body": lambda: (np.array([[0.1, 0.2, 0.3]], np.float32), np.ones(1, np.float32), 8),
    "leafcap-plus-one": lambda: (np.random.default_rng(48).uniform(0, 1, (17, 3)).astype(np.float32),
                                 np.ones(17, np.float32), 16),
    "leafcap-256": lambda: (np.random.default_rng(49).uniform(0, 1, (3000, 3)).astype(np.float32),
                            np.ones(3000, np.float32), 256),
    # 131,072 keys: the last size whose radix passes scan their digits inside
    # the scatter (128 tiles) and whose body-count scan is one block; one
    # more body takes the separate scan launches for both
    "plummer-131072": lambda: (workloads.plummer_sphere(131072, seed=50).pos,
                               workloads.plummer_sphere(131072, seed=50).mass, 16),
    "plummer-131073": lambda: (workloads.plummer_sphere(131073, seed=50).pos,
                               workloads.plummer_sphere(131073, seed=50).mass, 16),
    "disk2d-131073": lambda: (workloads.gaussian_disk(131073, seed=51).pos,
                              workloads.gaussian_disk(131073, seed=51).mass, 16),
    # one key past the sizes where the body sort's tiles grow (2048 keys per
    # tile from 524,288 keys, 4096 from 1,048,576): 257 tiles, the last one
    # holding a single key (both level orders, about 4 cells per 16 bodies
    # expected, go in tiles of 1024 cells)
    "plummer-524289": lambda: (workloads.plummer_sphere(524289, seed=53).pos,
                               workloads.plummer_sphere(524289, seed=53).mass, 16),
    "plummer-1048577": lambda: (workloads.plummer_sphere(1048577, seed=54).pos,
                                workloads.plummer_sphere(1048577, seed=54).mass, 16),
    # from 2^21 keys the radix passes rank each 4096-key tile in LDS before
    # writing it: a ragged last tile (2,848 keys) with the clumped, skewed
    # digits of the clustered mixture, and one key past the threshold in 2D
    "clustered-2100000": lambda: (workloads.clustered(2_100_000, seed=52).pos,
                                  workloads.clustered(2_100_000, seed=52).mass, 16),
    "disk2d-2097153": lambda: (workloads.gaussian_disk(2_097_153, seed=53).pos,
                               workloads.gaussian_disk(2_097_153, seed=53).mass, 16),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_tree_bit_exact(name):
    pos, mass, lc = CASES[name]()
    print(f"case {name} n={len(pos)} leaf_cap={lc}", flush=True)
    g = gpu_tree(pos, mass, lc)
    assert g["status"] == 0
    t = oracle.Tree(pos.astype(np.float64), np.asarray(mass, np.float64), lc)
    assert_tree_equal(g, t)


def test_nonfinite_is_sticky_until_next_build():
    from paper_1211_2293_amd import treecode
    pos = np.random.default_rng(50).uniform(0, 1, (1000, 3)).astype(np.float32)
    mass = np.ones(1000, np.float32)
    bad = pos.copy()
    bad[17, 1] = np.nan
    g = gpu_tree(bad, mass, 8, theta=0.5, eps=1e-2)
    assert g["status"] == treecode.TC_ENONFINITE
    tc = g["tc"]
    import torch
    tc.build(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda())
    assert tc.status() == treecode.TC_OK
    m = mass.copy()
    m[3] = -1.0
    g2 = gpu_tree(pos, m, 8)
    assert g2["status"] == treecode.TC_ENONFINITE


@pytest.mark.parametrize("dim", [3, 2])
def test_context_reuse_with_a_deeper_tree(dim):
    """A context shapes its moments launches by the level sizes of an
    earlier tree; the deepest small levels go to one single-block pass.  A
    shallow tree first, then a much deeper one (two tight clumps), then the
    shallow one again: every tree is still bit-exact."""
    import torch

    from paper_1211_2293_amd import treecode
    rng = np.random.default_rng(51)
    shallow = rng.uniform(0, 1, (4000, dim)).astype(np.float32)
    deep = _two_clumps(3000)[:, :dim].copy()
    deep[:50] = rng.uniform(0, 1, (50, dim))
    tc = treecode.Treecode(dim, leaf_cap=8)
    for pos in (shallow, deep, deep, shallow):
        mass = np.ones(len(pos), np.float32)
        g = gpu_tree(pos, mass, 8, tc=tc)
        torch.cuda.synchronize()
        assert g["status"] == treecode.TC_OK
        t = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), 8)
        print(f"dim={dim} n={len(pos)} depth {int(g['cells']['level'].max())}", flush=True)
        assert_tree_equal(g, t)


@pytest.mark.parametrize("dim", [3, 2])
def test_context_reuse_when_the_top_levels_no_longer_fit_in_lds(dim):
    """Two tight clumps far apart have a long chain of one or two cells per
    level at the top (levels 0..14 in 3D hold under 512 cells), so the next
    moments pass keeps those levels in LDS; a centrally concentrated tree
    built next holds over 17,000 cells there, and the pass must read the
    children from memory instead.  Then the clumps again.  All bit-exact."""
    import torch

    from paper_1211_2293_amd import treecode
    rng = np.random.default_rng(52)
    a = rng.normal(0.0, 1e-4, (50000, dim))
    b = rng.normal(1.0, 1e-4, (50000, dim))
    clumps = np.concatenate([a, b]).astype(np.float32)
    w = workloads.plummer_sphere(100000, seed=53) if dim == 3 else workloads.gaussian_disk(100000, seed=53)
    spread = np.asarray(w.pos, np.float32)
    tc = treecode.Treecode(dim, leaf_cap=16)
    for name, pos in (("clumps", clumps), ("spread", spread), ("clumps", clumps)):
        mass = np.ones(len(pos), np.float32)
        print(f"dim={dim} {name} n={len(pos)}", flush=True)
        g = gpu_tree(pos, mass, 16, tc=tc)
        torch.cuda.synchronize()
        assert g["status"] == treecode.TC_OK
        t = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), 16)
        assert_tree_equal(g, t)


def _strata_draw(n, buckets, per):
    """The bodies that the body sort samples: one at a hashed place of each of
    buckets x per equal strata."""
    S = buckets * per
    j = np.arange(S, dtype=np.uint64)
    lo, hi = j * n // S, (j + 1) * n // S
    m32 = np.uint64(0xffffffff)
    h = (j * np.uint64(2654435761)) & m32
    h ^= h >> np.uint64(15)
    h = (h * np.uint64(2246822519)) & m32
    h ^= h >> np.uint64(13)
    return (lo + h % (hi - lo)).astype(np.int64)


def _missed_by_the_draw(n, buckets, per, dim):
    """Bodies outside the sample all follow the sampled ones in key order, so
    one bucket holds nearly all of them (more than a block sorts in LDS)."""
    rng = np.random.default_rng(55)
    pos = rng.uniform(0.75, 1.0, (n, dim))
    pos[rng.permutation(n)[: n // 3]] = 0.875       # and many equal keys among them
    at = _strata_draw(n, buckets, per)
    pos[at] = rng.uniform(0.0, 0.25, (len(at), dim))
    return pos.astype(np.float32)


SORT_CASES = {
    # the rank sort's own sizes: one block, a partial block, a chunk of keys
    # and one more, its largest; then the first size with buckets
    **{f"n{n}": (lambda n=n: workloads.plummer_sphere(n, seed=56).pos) for n in
       (31, 32, 33, 4096, 4097, 8192, 8193, 16384, 16385, 65536, 65537, 262144, 262145, 524288, 1048577, 2097151)},
    "f64-262145": lambda: workloads.plummer_sphere(262145, seed=57).pos.astype(np.float64) * 1.1,
    "disk-300001": lambda: workloads.gaussian_disk(300001, seed=58).pos,
    "sorted-input": lambda: np.sort(workloads.plummer_sphere(40001, seed=59).pos, axis=0),
    "equal-30000": lambda: np.full((30000, 3), 0.5, np.float32),
    "few-places": lambda: np.random.default_rng(60).integers(0, 3, (50000, 3)).astype(np.float32),
    "missed-20000": lambda: _missed_by_the_draw(20000, 128, 4, 3),
    "missed-2d": lambda: _missed_by_the_draw(60000, 256, 4, 2),
}


@pytest.mark.parametrize("name", list(SORT_CASES))
def test_body_order_is_the_stable_order_of_the_keys(name):
    """The order by (key, input index) on both sides of every size where the
    body sort changes its shape, for equal keys and for inputs that its sample
    misses: keys and permutation against numpy's stable sort of the oracle's
    keys (equal whole numbers), and the bodies they gather."""
    pos = SORT_CASES[name]()
    n, dim = pos.shape
    mass = np.random.default_rng(61).uniform(0.5, 2.0, n).astype(pos.dtype)
    from paper_1211_2293_amd import treecode
    from tests.gpu_util import to_dev
    tc = treecode.Treecode(dim, leaf_cap=256)
    keep = (to_dev(pos), to_dev(mass))
    tc.build(*keep)
    assert tc.status() == treecode.TC_OK
    k, perm = tc.keys()
    k, perm = k.cpu().numpy().view(np.uint64), perm.cpu().numpy().view(np.uint32)
    lo, size = tc.root()
    L = 21 if dim == 3 else 31
    x = pos.astype(np.float64)
    np.testing.assert_array_equal(lo, x.min(0))
    q = np.minimum(np.floor((x - lo) * (2.0 ** L / size)), 2.0 ** L - 1).astype(np.uint64)
    key = np.zeros(n, np.uint64)
    for b in range(L):
        for a in range(dim):
            key |= ((q[:, a] >> np.uint64(b)) & np.uint64(1)) << np.uint64(dim * b + dim - 1 - a)
    want = np.argsort(key, kind="stable")
    np.testing.assert_array_equal(perm, want)
    np.testing.assert_array_equal(k, key[want])
    # the root's mass and centre are sums over the gathered bodies
    tc.moments()
    c = tc.cells()
    m = mass.astype(np.float64)
    assert abs(float(c["M"][0]) - m.sum()) <= 1e-12 * m.sum()
    com = (m[:, None] * x).sum(0) / m.sum()
    np.testing.assert_allclose(c["com"][0].cpu().numpy(), com, rtol=0, atol=1e-10 * np.abs(x).max())


@pytest.mark.parametrize("dim,n,lc", [(3, 150, 1), (3, 9000, 256), (3, 44_000, 1), (3, 46_000, 1), (3, 250_000, 1),
                                      (3, 380_000, 1), (2, 60_000, 1), (2, 270_000, 1), (3, 131_071, 1),
                                      (3, 131_072, 1), (2, 650, 1), (3, 1023, 1), (3, 1025, 2)])
def test_moments_on_both_sides_of_each_shape(dim, n, lc):
    """Cell moments and topology bit for bit against the oracle where the
    moments pass changes its shape: no cells above the blocks' subtrees, subtrees
    of 128 and of 256 cells, more cells above them than one block looks up in
    advance, and the levels above in launches of their own; and where the
    topology does: its scans folded in (up to 131,071 bodies with leaf_cap 1)
    and as launches, one tile of cells and a few."""
    pos = (workloads.plummer_sphere(n, seed=62).pos if dim == 3 else workloads.gaussian_disk(n, seed=63).pos)
    mass = np.random.default_rng(64).uniform(0.5, 2.0, n).astype(np.float32)
    g = gpu_tree(pos, mass, lc)
    assert g["status"] == 0
    assert_tree_equal(g, oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), lc))


@pytest.mark.parametrize("dim,sizes", [(3, (1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 65, 257, 3001)), (2, (1, 3, 4, 5, 8, 65, 257, 3001))])
def test_moments_of_leaves_of_every_remainder(dim, sizes):
    """Leaves of coincident places, each of the given number of bodies (beyond
    leaf_cap at the deepest level): masses, centres and quadrupoles bit for bit
    against the oracle, which sums a leaf's bodies in order."""
    rng = np.random.default_rng(65)
    at = rng.uniform(-1.0, 1.0, (len(sizes), dim))
    # a cloud below the resolution of the deepest level around each place
    pos = np.concatenate([a + rng.uniform(0.0, 2.0 ** -30 if dim == 3 else 2.0 ** -40, (s, dim))
                          for a, s in zip(at, sizes)])
    pos = pos[rng.permutation(len(pos))]
    mass = rng.uniform(0.5, 2.0, len(pos))
    g = gpu_tree(pos, mass, 1)
    assert g["status"] == 0
    t = oracle.Tree(pos, mass, 1)
    assert_tree_equal(g, t)
    assert g["cells"]["count"][g["cells"]["leaf"] == 1].max() > 2000


@pytest.mark.parametrize("dim,n", [(3, 380000), (2, 270000)])
@pytest.mark.parametrize("case", ["shallow", "deep", "deepest", "one place"])
def test_moments_wherever_the_levels_lie(dim, n, case):
    """Trees of a size that has the moments of the levels with the most cells
    in launches of their own (2^22 cell slots and more), with these levels near the
    root, in the middle, at the deepest level, and with no such level at all."""
    rng = np.random.default_rng(67)
    pos = rng.uniform(-1.0, 1.0, (n, dim))
    if case == "deep":
        pos[8:] *= 1e-4
    elif case == "deepest":                           # pairs that no cell parts
        pos[1::2] = pos[::2]
    elif case == "one place":
        pos[8:] = pos[8]
    mass = rng.uniform(0.5, 2.0, n)
    g = gpu_tree(pos, mass, 1)
    assert g["status"] == 0
    assert_tree_equal(g, oracle.Tree(pos, mass, 1))


@pytest.mark.parametrize("n,buckets,per,dim,dtype", [
    (20000, 128, 4, 3, np.float64), (100000, 256, 4, 3, np.float32), (100000, 256, 4, 3, np.float64),
    (100000, 256, 4, 2, np.float64), (150001, 256, 8, 2, np.float32), (270000, 512, 8, 3, np.float32)])
def test_a_bucket_beyond_lds_in_every_kernel(n, buckets, per, dim, dtype):
    """Inputs that the sample misses put nearly all bodies in one bucket, which
    is sorted in memory: by the kernel of the small and of the large buckets,
    for records of FP32 and FP64 bodies.  The stable order of the keys, and the
    bodies themselves (by the leaves' moments)."""
    pos = _missed_by_the_draw(n, buckets, per, dim).astype(dtype)
    mass = np.random.default_rng(66).uniform(0.5, 2.0, n).astype(dtype)
    g = gpu_tree(pos, mass, 16)
    assert g["status"] == 0
    t = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64), 16)
    assert_tree_equal(g, t)
