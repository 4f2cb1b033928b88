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
    most tile borders of the box fit cross dozens of nodes, and 64 tiles
    list more of them (about 1700) than a workgroup of the second level keeps in
    LDS (1536)."""
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
# smallest second group, a third level of one workgroup
@pytest.mark.parametrize("n,kind", [(512, "uniform"), (513, "uniform"), (1025, "dup"), (32768, "uniform"),
                                    (32769, "uniform"), (65537, "comb"), (100_000, "comb")])
def test_boxes_of_nodes_across_tiles(ctx, n, kind):
    pts = combs(n, 5) if kind == "comb" else W.small_random(n, 3, 5, kind)
    print(f"case boxes n={n} {kind}", flush=True)
    left, right, lo, hi, root = ctx.test_tree_boxes(torch.from_numpy(pts).cuda())
    mn, mx = node_boxes(pts, left.cpu().numpy(), right.cpu().numpy(), root)
    np.testing.assert_array_equal(lo.cpu().numpy(), mn)
    np.testing.assert_array_equal(hi.cpu().numpy(), mx)
