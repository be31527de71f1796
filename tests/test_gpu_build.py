"""The scene build at the sizes where its launches change: runs of leaves over
one or more blocks, the collapse by one block or by wavefronts of a second
launch, prefix sums by one block or three launches.  Both hierarchies are
checked level by level against the leaf boxes, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2607_22780_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


def check_tree(child, boxes, leaf_boxes):
    """child [m, w] (>= 0 node, < 0 leaf -(p + 1), 0x7fffffff none), boxes
    [m, w, 6] of the children: every node and leaf once, boxes their unions."""
    m, n = len(child), len(leaf_boxes)
    levels, front = [], np.array([0])
    seen_node, seen_leaf = np.zeros(m, int), np.zeros(n, int)
    while len(front):
        levels.append(front)
        seen_node[front] += 1
        c = child[front].ravel()
        np.add.at(seen_leaf, -c[c < 0] - 1, 1)
        front = c[(c >= 0) & (c != 0x7fffffff)]
    assert np.all(seen_node == 1) and np.all(seen_leaf == 1)
    own = np.full((m, 6), np.nan, np.float32)
    for front in reversed(levels):
        c = child[front]
        none = c == 0x7fffffff
        want = np.where((c < 0)[..., None], leaf_boxes[np.where(c < 0, -c - 1, 0)],
                        own[np.where((c >= 0) & ~none, c, 0)])
        np.testing.assert_array_equal(boxes[front][~none], want[~none])
        lo = np.where(none[..., None], np.inf, want[..., :3]).min(1)
        hi = np.where(none[..., None], -np.inf, want[..., 3:]).max(1)
        own[front] = np.concatenate([lo, hi], 1)


@pytest.mark.parametrize("n", [2, 3, 7, 511, 512, 513, 1025, 4096, 4097, 4099, 24576, 24577, 262145])
def test_hierarchies(grt_ctx, n):
    grt, ctx = grt_ctx
    from gpu_util import scene_tensors
    s = W.scene0(n=n, seed=2)
    if n == 4099:
        s.means[: n // 2] = s.means[0]  # equal codes: ties by position
    scene = grt.Scene(ctx, *scene_tensors(s))
    scene.build()  # again, over what the first build left
    torch.cuda.synchronize()
    a = {k: v.cpu().numpy() for k, v in scene.arrays().items()}
    nd = a["nodes"]
    check_tree(nd[:, 12:14].view(np.int32), nd[:, :12].reshape(n - 1, 2, 6), a["leaf_boxes"])
    wide = a["nodes4"][: int(a["nodes4_count"][0])]
    check_tree(wide[:, 24:28].view(np.int32), wide[:, :24].reshape(-1, 6, 4).transpose(0, 2, 1), a["leaf_boxes"])
    ids = a["order"]
    assert np.array_equal(np.sort(ids), np.arange(n))
    lo, hi = s.means.min(0), s.means.max(0)
    q = np.clip(np.floor((s.means - lo) / (hi - lo) * np.float32(1024.0)).astype(np.int64), 0, 1023)
    code = np.zeros(n, np.int64)
    for b in range(10):
        for k in range(3):
            code |= ((q[:, k] >> b) & 1) << (3 * b + 2 - k)
    np.testing.assert_array_equal(ids, np.argsort(code, kind="stable"))
