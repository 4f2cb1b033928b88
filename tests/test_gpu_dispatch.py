"""Edges of the kernels' tiles and of the rules that choose between them,
through the C ABI, against the CPU oracle or a plain definition."""
import numpy as np
import pytest

import oracle
from paper_2207_00514_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2207_00514_amd as emst
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    return emst.Context(0)


def combs(n, seed):
    """Cells of a 16^3 grid, each with 60 points at its corner and a
    geometric comb of 48 points that halves its offset along one axis after
    the other: the radix tree nests about 48 nodes around every corner, so
    most tile borders cross dozens of nodes, and 64 tiles leave more of
    them (about 1700) than a workgroup of the second level takes at a time
    (1024)."""
    rng = np.random.default_rng(seed)
    corner = rng.permutation(16 ** 3)[:-(-n // 108)]
    corner = np.stack([corner % 16, corner // 16 % 16, corner // 256], 1) / 16.0
    step = np.arange(48)
    off = np.zeros((108, 3))
    off[step, step % 3] = 2.0 ** -(5 + step // 3)
    pts = (corner[:, None, :] + off[None, :, :]).reshape(-1, 3)[:n]
    return np.ascontiguousarray(pts[rng.permutation(n)].astype(np.float32))


def node_boxes(pts, left, right, root):
    n = len(pts)
    mn, mx = np.zeros((n - 1, 3), np.float32), np.zeros((n - 1, 3), np.float32)
    order, stack = [], [root]
    while stack:
        k = stack.pop()
        order.append(k)
        stack += [c for c in (left[k], right[k]) if c >= 0]
    for k in reversed(order):
        box = [(pts[-c - 1], pts[-c - 1]) if c < 0 else (mn[c], mx[c]) for c in (left[k], right[k])]
        mn[k], mx[k] = np.minimum(box[0][0], box[1][0]), np.maximum(box[0][1], box[1][1])
    assert len(order) == n - 1
    return mn, mx


# tiles of 512 leaves, groups of 64 tiles: one tile, two, one full group, the
# smallest second group, a third level of one workgroup; whole tiles below one node
@pytest.mark.parametrize("n,kind", [(512, "uniform"), (513, "uniform"), (1025, "dup"), (32768, "uniform"),
                                    (32769, "uniform"), (65537, "comb"), (100_000, "comb"),
                                    (1024, "same"), (40_000, "same")])
def test_boxes_of_nodes_across_tiles(ctx, n, kind):
    pts = combs(n, 5) if kind == "comb" else W.identical(n) if kind == "same" else W.small_random(n, 3, 5, kind)
    print(f"case boxes n={n} {kind}", flush=True)
    left, right, lo, hi, root = ctx.test_tree_boxes(torch.from_numpy(pts).cuda())
    mn, mx = node_boxes(pts, left.cpu().numpy(), right.cpu().numpy(), root)
    np.testing.assert_array_equal(lo.cpu().numpy(), mn)
    np.testing.assert_array_equal(hi.cpu().numpy(), mx)


def solve(ctx, pts):
    e, w, d2 = ctx.build(torch.from_numpy(np.ascontiguousarray(pts, np.float32)).cuda())
    torch.cuda.synchronize()
    return e.cpu().numpy(), w.cpu().numpy(), d2.cpu().numpy()


def assert_tree(got, ref, tag):
    e, w, d2 = got
    assert np.array_equal(e, ref.edges), f"{tag}: edges differ"
    assert np.array_equal(d2.view(np.uint32), ref.d2.view(np.uint32)), f"{tag}: d2 differ"
    assert np.array_equal(w.view(np.uint32), ref.w.view(np.uint32)), f"{tag}: weights differ"


# Clouds solved without a tree: one tile of 64 points and its edges, several
# tiles, the largest cloud merged by one workgroup and the first one merged
# by many, the largest such cloud and the first one with a tree
FLAT = [2, 3, 63, 64, 65, 129, 1000, 4095, 4096, 4097, 16383, 16384, 16385]


@pytest.mark.parametrize("kind", ["uniform", "int", "dup", "outlier"])
@pytest.mark.parametrize("n", FLAT)
def test_clouds_without_a_tree(ctx, n, kind):
    for dim in (2, 3):
        pts = W.small_random(n, dim, n + dim, kind)
        print(f"case flat n={n} dim={dim} {kind}", flush=True)
        got = solve(ctx, pts)
        assert (ctx.stats()["traversal_variant"] == -1) == (n <= 16384)
        assert_tree(got, oracle.emst(pts, threads=8), f"{kind} n={n} dim={dim}")


def growing_gaps(n):
    """Every point's nearest neighbour is its predecessor: one chain of n
    successors in the first merge."""
    x = np.cumsum(1.0 + np.arange(n) * 1e-3)
    return np.stack([x, np.zeros(n)], 1)[np.random.default_rng(1).permutation(n)].astype(np.float32)


FLAT_FORMS = {
    "identical": W.identical(1000), "grid2d": W.integer_grid(100, 2, seed=1), "grid3d": W.integer_grid(27, 3, seed=2),
    "collinear": W.collinear(3000, 2, seed=3),
    "growing gaps": growing_gaps(12_000), "growing gaps 4k": growing_gaps(4000), "two clusters": W.two_clusters(2000, 3, seed=5),
    "skewed": W.make("skewed3d_2m", 10_000), "clustered": W.clustered3d(16_000, seed=6),
    "cosmology": W.cosmology3d(15_000, seed=7),
    "star": np.concatenate([np.zeros((1, 3)), np.eye(3), -np.eye(3)] * 2000).astype(np.float32),
    "denormal": (np.random.default_rng(3).random((500, 3)) * 1e-19).astype(np.float32),
    "large": (np.random.default_rng(4).random((500, 3)) * 1e18).astype(np.float32),
}


@pytest.mark.parametrize("name", sorted(FLAT_FORMS))
def test_forms_without_a_tree(ctx, name):
    pts = FLAT_FORMS[name]
    print(f"case flat {name}", flush=True)
    assert_tree(solve(ctx, pts), oracle.emst(pts, threads=8), name)


@pytest.mark.parametrize("n", [100, 20_000])
@pytest.mark.parametrize("bad", [np.nan, np.inf, 3e38])
def test_refused_clouds_write_nothing(ctx, n, bad):
    import paper_2207_00514_amd as emst
    pts = W.small_random(n, 3, 1)
    pts[n // 2, 1] = bad
    pts[n // 3, 1] = -3e38 if np.isfinite(bad) else 0.0
    out = (torch.full((n - 1, 2), 7, dtype=torch.int32, device="cuda"), torch.full((n - 1,), 7.0, device="cuda"),
           torch.full((n - 1,), 7.0, device="cuda"))
    with pytest.raises(emst.EmstError) as ei:
        ctx.build(torch.from_numpy(pts).cuda(), out=out)
    assert ei.value.name == ("EMST_ERANGE" if np.isfinite(bad) else "EMST_ENONFINITE")
    assert all(bool((t == 7).all()) for t in out)
    good = W.small_random(n, 3, 2)
    assert_tree(solve(ctx, good), oracle.emst(good, threads=8), "after a refused cloud")


def test_small_clouds_on_several_threads_and_streams():
    """Four threads with a context and a stream each: their workgroups share
    the device, so those of one search do not all run at once."""
    import threading
    import paper_2207_00514_amd as emst
    clouds = [W.clustered3d(16_384, seed=s) for s in range(4)] + [W.uniform2d(9_000, seed=s) for s in range(4)]
    refs = [oracle.emst(p, threads=8) for p in clouds]
    wrong = []

    def work(k):
        ctx, st = emst.Context(0), torch.cuda.Stream()
        with torch.cuda.stream(st):
            dev = [torch.from_numpy(p).cuda() for p in clouds]
            for rep in range(10):
                c = (k + rep) % len(clouds)
                e, w, d2 = ctx.build(dev[c], stream=st)
                st.synchronize()
                if not (np.array_equal(e.cpu().numpy(), refs[c].edges)
                        and np.array_equal(d2.cpu().numpy().view(np.uint32), refs[c].d2.view(np.uint32))):
                    wrong.append((k, rep, c))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


# one-launch passes on tiles of 2,048 keys below 2^19 keys, three launches above
@pytest.mark.parametrize("n", [3, 2047, 2048, 2049, 16_385, 65_537, 300_001, 524_287, 524_288])
def test_sort_sizes(ctx, n):
    rng = np.random.default_rng(n)
    keys = rng.integers(-2 ** 63, 2 ** 63, n, dtype=np.int64)
    keys[n // 2:] = rng.integers(0, 3, n - n // 2)  # most digits the same, many equal keys
    keys[rng.permutation(n)[: n // 4]] = -1
    vals = np.arange(n, dtype=np.int32)
    k, v = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()
    print(f"case sort n={n}", flush=True)
    ctx.test_radix_sort(k, v)
    order = np.argsort(keys.view(np.uint64), kind="stable")
    assert np.array_equal(k.cpu().numpy(), keys[order])
    assert np.array_equal(v.cpu().numpy(), vals[order])


# a look-back that does not wait for the tiles before it: passes on tiles of
# 2,048 keys (two, many and the most of them) and of 4,096
@pytest.mark.parametrize("n", [4096, 65_537, 524_287, 4_194_304])
def test_sort_whose_look_backs_do_not_wait(ctx, n):
    rng = np.random.default_rng(n + 1)
    keys = rng.integers(-2 ** 63, 2 ** 63, n, dtype=np.int64)
    keys[n // 2:] = rng.integers(0, 3, n - n // 2)
    vals = np.arange(n, dtype=np.int32)
    k, v = torch.from_numpy(keys).cuda(), torch.from_numpy(vals).cuda()
    print(f"case sort without waits n={n}", flush=True)
    counted = ctx.test_radix_sort_polls(k, v, 0)
    assert counted > 0 or n == 4096  # (one predecessor, which may have been done)
    order = np.argsort(keys.view(np.uint64), kind="stable")
    assert np.array_equal(k.cpu().numpy(), keys[order])
    assert np.array_equal(v.cpu().numpy(), vals[order])


def test_polled_memory_is_coherent(ctx):
    assert ctx.test_mirror_is_coherent()


# dense clouds (codes by rank) with an axis that all points, or many, share
SHARED_AXES = {"line": (150_000, lambda r, x: np.stack([x, 0.5 * x, 0.0 * x], 1), 0),
               "plane": (60_000, lambda r, x: np.stack([x, r.random(len(x)), 0.0 * x], 1), 1),
               "terraces": (60_000, lambda r, x: np.stack([x, r.random(len(x)), np.floor(8 * r.random(len(x)))], 1), 1)}


@pytest.mark.parametrize("name", sorted(SHARED_AXES))
def test_rank_codes_of_points_that_share_a_coordinate(ctx, name):
    n, make, far = SHARED_AXES[name]
    rng = np.random.default_rng(17)
    pts = make(rng, rng.random(n)).astype(np.float32)
    if far:
        pts[n // 2] = 2.0 ** 20  # every other point in one cell of the box
    print(f"case shared axis {name}", flush=True)
    assert_tree(solve(ctx, pts), oracle.emst(pts, threads=8), name)
    assert ctx.stats()["rank_codes"] == 1
    if name == "terraces":
        return
    # an axis without information costs a search nothing: in 2D, where codes of
    # 32 bits an axis hold the line's and the unit square's points apart, as many
    # boxes are tested up to a factor of 2 (5 times as many where the shared
    # coordinate's ranks follow the indices)
    ctx.set_counting(True)
    ctx.build(torch.from_numpy(pts).cuda())
    tests = ctx.stats()["child_tests"]
    ctx.build(torch.from_numpy(np.ascontiguousarray(pts[np.arange(n) != n // 2 if far else slice(None), :2])).cuda())
    plain = ctx.stats()["child_tests"]
    ctx.set_counting(False)
    assert tests <= 2 * plain, (tests, plain)


def core_reference(pts, k):
    """The k-th smallest D(i, j) over all j, float32 in the kernels' order."""
    n, out = len(pts), np.empty(len(pts), np.float32)
    for a in range(0, n, 256):
        s = np.zeros((min(256, n - a), n), np.float32)
        for c in range(pts.shape[1]):
            d = pts[a:a + 256, c][:, None] - pts[None, :, c]
            s = d * d if c == 0 else s + d * d
        out[a:a + 256] = np.partition(s, k - 1, axis=1)[:, k - 1]
    return out


# every list length (4, 8, 16, 32, 64) full and not, windows clipped at both
# ends of the cloud, duplicates, and denormal distances
@pytest.mark.parametrize("k", [2, 4, 5, 8, 9, 16, 17, 31, 32, 33, 64])
def test_core_distances_of_every_list_length(ctx, k):
    clouds = [W.small_random(max(k, 65), 3, 1), W.small_random(k, 2, 2), W.small_random(2500, 3, 3, "dup"),
              W.small_random(2500, 2, 4, "int"), W.clustered3d(3000, seed=5),
              (np.random.default_rng(6).random((1500, 3)) * 1e-20).astype(np.float32)]
    for n, pts in enumerate(clouds):
        print(f"case core k={k} cloud {n}", flush=True)
        got = ctx.core_distances(torch.from_numpy(pts).cuda(), k).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), core_reference(pts, k).view(np.uint32)), f"cloud {n}"


def test_runs_of_component_zero_beside_another(ctx):
    """The component labelled 0 with a run that starts at lane 1 of a wave
    (and at lanes 16, 32 and 63 of others): the offers and bounds of the lane
    before stay that lane's own."""
    n = 1000
    rng = np.random.default_rng(12)
    x = np.cumsum(1.0 + rng.random(n))
    zero = [0, 65, 66, 144, 145, 224, 319]  # sorted positions, the order along the line
    for p in zero[1:]:
        x[p - 1:] -= 0.9 * (x[p - 1] - x[p - 2])  # the lane before has the shortest edges around
    comp = np.arange(n)
    comp[zero] = 0
    pts = np.stack([x, np.zeros(n)], 1).astype(np.float32)
    d = (pts[1:, 0] - pts[:-1, 0]) ** 2
    nearest = np.full(n, np.inf, np.float32)  # per component: a point's nearest other-component point is a neighbour
    for k in range(n - 1):
        if comp[k] != comp[k + 1]:
            for c in (comp[k], comp[k + 1]):
                nearest[c] = min(nearest[c], d[k])
    for variant in (7, 13):
        print(f"case runs of component 0, variant {variant}", flush=True)
        r = ctx.test_round(torch.from_numpy(pts).cuda(), torch.from_numpy(comp.astype(np.int32)).cuda(), 1, variant)
        for name in ("comp_d2", "bound"):
            assert np.array_equal(r[name].cpu().numpy(), nearest[comp]), f"variant {variant}: {name}"


def check_batch(ctx, clouds):
    res = ctx.build_batched([torch.from_numpy(c).cuda() for c in clouds])
    torch.cuda.synchronize()
    for k, (c, (e, w, d2)) in enumerate(zip(clouds, res)):
        assert_tree((e.cpu().numpy(), w.cpu().numpy(), d2.cpu().numpy()), oracle.emst(c, threads=8), f"cloud {k}")


# waves of 64 points inside one cloud, across clouds and past the end; 2D and
# 3D; ties that need the in-place order and those that need the full one
@pytest.mark.parametrize("sizes", [[64, 64, 64], [1, 63, 64, 65, 2, 0, 127, 1], [1000, 1, 200, 5000, 64, 129],
                                   [40_000, 3, 30_000], [20_001]])
@pytest.mark.parametrize("kind", ["uniform", "int", "dup", "outlier"])
def test_batch_edge_order(ctx, sizes, kind):
    print(f"case batch {sizes} {kind}", flush=True)
    check_batch(ctx, [W.small_random(n, 2 + k % 2, 7 * k + n, kind) for k, n in enumerate(sizes)])


def test_batch_whose_order_needs_more_than_64_bits(ctx):
    """70,000 clouds (17 bits) with one of 70,000 points (17 bits): with the
    31 bits of D one more than a key holds, so the slots are sorted by cloud."""
    rng = np.random.default_rng(9)
    big = W.clustered3d(70_000, seed=9)
    pairs = rng.random((69_999, 2, 2)).astype(np.float32)
    clouds = [torch.from_numpy(big).cuda()] + list(torch.from_numpy(pairs).cuda())
    res = ctx.build_batched(clouds)
    torch.cuda.synchronize()
    e, w, d2 = (t.cpu().numpy() for t in res[0])
    assert_tree((e, w, d2), oracle.emst(big, threads=8), "the large cloud")
    edges = torch.cat([r[0] for r in res[1:]]).cpu().numpy()
    got = torch.cat([r[2] for r in res[1:]]).cpu().numpy()
    dx, dy = (pairs[:, 0] - pairs[:, 1]).T
    assert np.array_equal(edges, np.tile(np.array([[0, 1]], np.int32), (69_999, 1)))
    assert np.array_equal(got.view(np.uint32), (dx * dx + dy * dy).view(np.uint32))


# Tiles of the round kernels: 1, 2, 4 and 8 positions a thread up to 2^19, 2^20,
# 2^21 points and above, their partials in the sort's histogram below 8; up to
# 2,048 tiles (2^22 points) their scans are folded into the consumers
@pytest.mark.parametrize("n", [1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1, 1 << 22,
                               (1 << 22) + 1])
def test_tile_sizes_of_the_round_kernels(n):
    import paper_2207_00514_amd as emst
    ctx = emst.Context(0)
    ctx.set_traversal(13)
    pts = W.clustered3d(n, seed=33) if n <= 1 << 20 else W.uniform2d(n, seed=34)
    print(f"case tiles n={n}", flush=True)
    assert_tree(solve(ctx, pts), oracle.kdboruvka(pts, threads=16), f"n={n}")
    if n > 3 << 18:
        assert any(q < n for q in ctx.stats()["queries_round"][2:])  # query lists ran


# edges of equal length and equal smaller endpoint, which the order by (D, u)
# leaves to the in-place order by v: with a tree, by variant and by size
@pytest.mark.parametrize("dim,span", [(2, 6000), (3, 600)])
def test_short_runs_of_equal_lengths_with_a_tree(dim, span):
    import paper_2207_00514_amd as emst
    ctx = emst.Context(0)
    ties = 0
    for n, variant in [(3000, 13)] * 6 + [(20_000, -1)] * 2:
        rng = np.random.default_rng(500 + ties + n)
        pts = rng.integers(0, span * (1 if n == 3000 else 3), (n, dim)).astype(np.float32)
        ctx.set_traversal(variant)
        print(f"case ties n={n} dim={dim}", flush=True)
        ref = oracle.emst(pts, threads=8)
        assert_tree(solve(ctx, pts), ref, f"n={n} dim={dim}")
        assert ctx.stats()["traversal_variant"] == 13
        k = np.sort((ref.d2.view(np.uint32).astype(np.uint64) << np.uint64(32)) | ref.edges[:, 0].astype(np.uint64))
        ties += int((k[1:] == k[:-1]).sum())
    assert ties > 0


def test_every_build_of_several_threads():
    """Four threads with a context and a stream each, clouds with and without a
    tree: every build is made, none raises, and edges, lengths and weights are
    the oracle's."""
    import threading
    import paper_2207_00514_amd as emst
    clouds = [W.clustered3d(16_384, seed=1), W.uniform2d(9_000, seed=2), W.clustered3d(30_000, seed=3),
              W.small_random(20_001, 2, 4, "dup")]
    refs = [oracle.emst(p, threads=8) for p in clouds]
    done, wrong = [], []

    def work(k):
        try:
            ctx, st = emst.Context(0), torch.cuda.Stream()
            with torch.cuda.stream(st):
                dev = [torch.from_numpy(p).cuda() for p in clouds]
                for rep in range(12):
                    c = (k + rep) % len(clouds)
                    got = ctx.build(dev[c], stream=st)
                    st.synchronize()
                    e, w, d2 = (t.cpu().numpy() for t in got)
                    assert_tree((e, w, d2), refs[c], f"thread {k} build {rep}")
                    done.append((k, rep))
        except BaseException as exc:  # (a thread's exception fails no test by itself)
            wrong.append((k, repr(exc)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong and len(done) == 48, (wrong, len(done))
