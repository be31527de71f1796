"""Every hit-buffer size that the MIS render and its backward take, plain and with the
shading state's gradients, by re-traversal and from hit lists on both sides of
the length where the shading state's kernel changes, through rays with hundreds
of hits: the oracle's gradients, whichever kernel a size runs."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2607_22780_amd import workloads as W
from test_gpu_bench_path import stack_scene
from test_gpu_shading_grad import check13, check_shade, edge_pixels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    from gpu_util import scene_tensors, t
    from paper_2607_22780_amd import grt
    ctx = grt.Context(0)
    s = stack_scene()
    g = np.random.default_rng(8)
    n = 25
    x = np.zeros((n, 3), np.float32)
    x[:, 0::2] = g.uniform(-0.5, 0.5, (n, 2))
    wo = W.random_unit_vectors(g, n)
    wo[:, 1] = np.abs(wo[:, 1]) + 0.3
    wo = (wo / np.linalg.norm(wo, axis=1, keepdims=True)).astype(np.float32)
    gb = W.GBuffer(5, 5, x, np.tile(np.float32([0, 1, 0]), (n, 1)), wo, g.uniform(0, 1, (n, 3)).astype(np.float32),
                   g.uniform(0.05, 1, n).astype(np.float32), (g.uniform(0, 1, n) < 0.3).astype(np.float32),
                   np.ones(n, np.uint8))
    env, split = W.envmap(32, 64, seed=4), (4, 2, 2)
    clean = ~edge_pixels(O.render_mis(s, gb, env, split, 5, dump=True))
    assert clean.mean() > 0.5
    up = (g.normal(0, 1, (n, 3)) * clean[:, None]).astype(np.float32)
    ref = O.render_mis_backward(s, gb, env, split, 5, up, with_abs=True, shading=True)
    scene, E = grt.Scene(ctx, *scene_tensors(s)), grt.Env(ctx, t(env))
    return grt, scene, E, grt.GBuffer.from_numpy(gb, torch.device("cuda", 0)), split, t(up), ref


@pytest.mark.parametrize("k", [1, 2, 4, 8, 12, 13, 16, 32])
@pytest.mark.parametrize("cap", [0, 31, 32, 400])
def test_backward_at_every_size(case, k, cap):
    grt, scene, E, G, split, up, (r13, r13_abs, rsh, rsh_abs) = case
    hits = grt.make_hit_list(G.npix, sum(split), cap, up.device) if cap else None
    lists = dict(split=split, seed=5, hits=hits, hit_cap=cap)
    fwd = grt.render_mis(scene, E, G, k=8, save=True, **lists)
    if cap:
        count = hits[: G.npix * sum(split)].cpu().numpy()
        assert (count > cap).any() == (cap < 400)
    if k != 13:  # (the backward's alone)
        own = grt.render_mis(scene, E, G, k=k, save=True, **lists)
        np.testing.assert_allclose(own["rgb"].cpu().numpy(), fwd["rgb"].cpu().numpy(), rtol=1e-5, atol=1e-6)
    plain = grt.render_mis_backward(scene, E, G, up, fwd["saved"], k=k, **lists)
    shaded, state = grt.render_mis_backward_shading(scene, E, G, up, fwd["saved"], k=k, **lists)
    torch.cuda.synchronize()
    for grads in (plain, shaded):
        check13({name: v.cpu().numpy() for name, v in grads.items()}, r13, r13_abs)
    check_shade(state, rsh, rsh_abs)
