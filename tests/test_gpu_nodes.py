"""The quantized nodes the traversal loads never lose a hit: scenes at other
scales and away from the origin, flat ones whose boxes are only their padding
thick, rays along the axes, and a surfel whose parameters are NaN.  Hit lists
are compared bit for bit with the brute-force oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2607_22780_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


def flat_scene(n, seed, size, at):
    """Surfels on three walls through the point (at, at, at), axis-aligned."""
    g = np.random.default_rng(seed)
    axis = g.integers(0, 3, n)
    p = g.uniform(-1.0, 1.0, (n, 3)) * size
    p[np.arange(n), axis] = 0.0
    nrm = np.eye(3)[axis] * g.choice([-1.0, 1.0], n)[:, None]
    q = W.quats_aligned_to(nrm, g.uniform(0, 2 * np.pi, n))
    f = lambda a: np.ascontiguousarray(a, np.float32)
    return W.Surfels(f(p + at), f(g.uniform(0.02, 0.1, (n, 2)) * size), f(q), f(g.uniform(0.2, 0.99, n)),
                     f(g.uniform(0, 1, (n, 3))))


def rays_at(g, m, size, at):
    o = (g.uniform(-1.0, 1.0, (m, 3)) * size + at).astype(np.float32)
    d = W.random_unit_vectors(g, m)
    d[: m // 4] = np.eye(3)[g.integers(0, 3, m // 4)] * g.choice([-1.0, 1.0], m // 4)[:, None]  # along the axes
    d[m // 4: m // 2, 0] *= 1e-6  # nearly across one
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return o, d.astype(np.float32)


def check(grt, ctx, s, o, d, keep=None):
    from gpu_util import scene_tensors, t
    ref = O.trace(s if keep is None else s.subset(keep), o, d, cap=48)
    scene = grt.Scene(ctx, *scene_tensors(s))
    for k in (1, 16):
        out = grt.trace(scene, t(o), t(d), k=k, dump_cap=48)
        torch.cuda.synchronize()
        ok = ref["margins"][:, 3] >= 1e-5
        ids = ref["ids"] if keep is None else np.where(ref["ids"] >= 0, keep[ref["ids"]], -1)
        np.testing.assert_array_equal(out["nhit"].cpu().numpy()[ok], ref["nhit"][ok])
        np.testing.assert_array_equal(out["ids"].cpu().numpy()[ok], ids[ok])
        np.testing.assert_array_equal(out["tau"].cpu().numpy()[ok].view(np.uint32), ref["tau"][ok].view(np.uint32))
    assert ref["nhit"].sum() > 0


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 17, 2000])
@pytest.mark.parametrize("size,at", [(1.0, 0.0), (0.05, 0.0), (30.0, 0.0), (1.0, 7.0), (1.0, -60.0)])
def test_scaled_and_moved_scenes(grt_ctx, n, size, at):
    grt, ctx = grt_ctx
    g = np.random.default_rng([n, 5])
    o, d = rays_at(g, 600, size, at)
    check(grt, ctx, flat_scene(n, n, size, at), o, d)
    s = W.scene0(n=n, seed=3)
    w = W.Surfels(np.float32(s.means * size + at), np.float32(s.scales * 4 * size), s.quats, s.opacity, s.rgb)
    check(grt, ctx, w, o, d)


def test_nan_surfels_are_no_hits(grt_ctx):
    grt, ctx = grt_ctx
    s = W.scene0(n=700, seed=4)
    s.scales[:] *= 3.0
    bad = np.arange(5, 700, 37)
    s.means[bad[0::3]] = np.nan
    s.scales[bad[1::3]] = np.nan
    s.quats[bad[2::3]] = 0.0
    keep = np.setdiff1d(np.arange(700), bad)
    g = np.random.default_rng(6)
    o, d = rays_at(g, 800, 1.0, 0.0)
    check(grt, ctx, s, o, d, keep)


@pytest.mark.parametrize("size,at,dist", [(300.0, 0.0, 1.0), (1000.0, 0.0, 1.0), (1.0, 300.0, 2.0),
                                          (0.2, -1000.0, 2.0), (1.0, 0.0, 1000.0)])
def test_far_scenes(grt_ctx, size, at, dist):
    """Coordinates and depths where the boxes' padding is below a unit in the
    last place; rays aimed at the surfels from `dist` sizes away."""
    grt, ctx = grt_ctx
    g = np.random.default_rng(8)
    target = g.uniform(-1.0, 1.0, (2000, 3)) * size + at
    o = (target + W.random_unit_vectors(g, 2000) * size * dist * g.uniform(0.5, 1.0, (2000, 1))).astype(np.float32)
    d = target - o
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    s = W.scene0(n=2000, seed=3)
    check(grt, ctx, W.Surfels(np.float32(s.means * size + at), np.float32(s.scales * 4 * size), s.quats, s.opacity,
                              s.rgb), o, d)
