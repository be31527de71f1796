"""The clustered hierarchy at its edges: blocks of 512 clusters, launches that
leave an eighth, and the bound on its height that the walks' stacks need."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


def scene_of(kind, n):
    """means, scales, quats, opacity, rgb."""
    g = np.random.default_rng(n)
    means = g.uniform(-1, 1, (n, 3))
    size = np.full(n, 0.02)
    if kind == "same":  # every pair equally close
        means[:] = means[0]
    elif kind == "chain":  # each surfel far larger than all before it: free merges would nest them one by one
        size = 1e-6 * 1.04 ** (np.arange(n) % 500)
        means = np.stack([size * 3.0, 0 * size, 0 * size], 1)
    elif kind == "endless":  # no closest pair
        size[n // 3 : 2 * n // 3] = np.inf
    q = g.normal(size=(n, 4))
    f = lambda a: np.ascontiguousarray(a, np.float32)
    return [f(means), f(np.stack([size, size], 1)), f(q / np.linalg.norm(q, axis=1, keepdims=True)),
            f(g.uniform(0.3, 0.9, n)), f(g.uniform(0, 1, (n, 3)))]


@pytest.mark.parametrize("n", [2, 64, 65, 511, 512, 513, 4096, 4097, 33_000])
@pytest.mark.parametrize("kind", ["scatter", "same", "chain", "endless"])
def test_height_and_order(grt_ctx, kind, n):
    """Every node and leaf has one parent, which has a lower number (so the
    tree is one); no path is longer than 63 edges; leaf counts add up."""
    import torch
    grt, ctx = grt_ctx
    scene = grt.Scene(ctx, *[torch.from_numpy(a).cuda() for a in scene_of(kind, n)])
    torch.cuda.synchronize()
    nd = scene.arrays()["nodes"].cpu().numpy().view(np.int32)
    ch, count = nd[:, 12:14], nd[:, 14]
    parent = np.repeat(np.arange(n - 1), 2).reshape(n - 1, 2)
    inner = ch >= 0
    np.testing.assert_array_equal(np.sort(ch[inner]), np.arange(1, n - 1))
    np.testing.assert_array_equal(np.sort(-ch[~inner] - 1), np.arange(n))
    assert np.all(ch[inner] > parent[inner])
    high = np.zeros(n - 1, int)
    for i in range(n - 2, -1, -1):
        high[i] = 1 + max(high[c] if c >= 0 else 0 for c in ch[i])
        assert count[i] == sum(count[c] if c >= 0 else 1 for c in ch[i])
    assert high[0] <= 63
