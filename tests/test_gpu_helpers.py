"""Compositing by helper lanes: numbers of rays that composite at once on both
sides of 16 and 32 (four, two or one helper each) and buffers shorter than the
helpers of a ray.  Copies of one ray reach every step together."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from test_gpu_bench_path import check_grads, stack_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


@pytest.mark.parametrize("same", [True, False])
@pytest.mark.parametrize("nr", [1, 3, 15, 16, 17, 31, 32, 33, 63, 64])
def test_compositing_lanes(grt_ctx, nr, same):
    grt, ctx = grt_ctx
    from gpu_util import scene_tensors, t
    n = 37
    s = stack_scene(nstack=n, alpha=0.05)
    g = np.random.default_rng(nr)
    o = np.zeros((nr, 3), np.float32)
    o[:, 0::2] = g.uniform(-0.5, 0.5, (1 if same else nr, 2))
    d = g.standard_normal((1 if same else nr, 3)) * 0.3
    d[:, 1] = 1.0
    d = np.repeat((d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32), nr if same else 1, axis=0)
    ref = O.trace(s, o, d, cap=n)
    ok = ref["margins"][:, 3] >= 1e-5
    assert np.all(ref["nhit"] == n)
    scene = grt.Scene(ctx, *scene_tensors(s))
    gC = (g.standard_normal((nr, 3)) * ok[:, None]).astype(np.float32)
    gT = (g.standard_normal(nr) * ok).astype(np.float32)
    want = O.trace_backward(s, o, d, gC, gT, with_abs=True)
    for k in (1, 2, 4, 8, 16, 32):
        out = grt.trace(scene, t(o), t(d), k=k, dump_cap=n)
        grads = grt.trace_backward(scene, t(o), t(d), out["rgb"], out["T"], t(gC), t(gT), k=k)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out["ids"].cpu().numpy()[ok], ref["ids"][ok])
        np.testing.assert_array_equal(out["tau"].cpu().numpy()[ok].view(np.uint32), ref["tau"][ok].view(np.uint32))
        np.testing.assert_allclose(out["rgb"].cpu().numpy()[ok], ref["C"][ok], rtol=1e-4, atol=1e-5)
        np.testing.assert_allclose(out["T"].cpu().numpy()[ok], ref["T"][ok], rtol=1e-4, atol=1e-5)
        check_grads({kk: v.cpu().numpy() for kk, v in grads.items()}, want)
