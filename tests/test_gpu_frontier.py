"""The traversal's stacks where their windows fill, empty and wrap: rays
through stacks of low-opacity surfels, as many as a window of the walk stack
or the deferred list holds, a few more, a few less, and around the length at
which the deferred list is dropped.  Hit lists are compared bit for bit with
the oracle, gradients to the backward's bar."""
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


@pytest.mark.parametrize("n", [9, 17, 20, 25, 28, 33, 41, 64, 177, 193, 201, 230])
def test_stack_windows(grt_ctx, n):
    grt, ctx = grt_ctx
    from gpu_util import scene_tensors, t
    s = stack_scene(nstack=n, alpha=0.02)
    g = np.random.default_rng(n)
    nr = 67
    o = np.zeros((nr, 3), np.float32)
    o[:, 0::2] = g.uniform(-0.5, 0.5, (nr, 2))
    d = g.standard_normal((nr, 3)) * 0.3
    d[:, 1] = 1.0
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    ref = O.trace(s, o, d, cap=n)
    ok = ref["margins"][:, 3] >= 1e-5
    assert ok.mean() > 0.95 and np.all(ref["nhit"] == n)
    scene = grt.Scene(ctx, *scene_tensors(s))
    gC = (g.standard_normal((nr, 3)) * ok[:, None]).astype(np.float32)
    gT = (g.standard_normal(nr) * ok).astype(np.float32)
    want = O.trace_backward(s, o, d, gC, gT, with_abs=True)
    for k in (1, 4, 12, 16):
        out = grt.trace(scene, t(o), t(d), k=k, dump_cap=n)
        grads = grt.trace_backward(scene, t(o), t(d), out["rgb"], out["T"], t(gC), t(gT), k=k)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out["nhit"].cpu().numpy()[ok], ref["nhit"][ok])
        np.testing.assert_array_equal(out["ids"].cpu().numpy()[ok], ref["ids"][ok])
        np.testing.assert_array_equal(out["tau"].cpu().numpy()[ok].view(np.uint32), ref["tau"][ok].view(np.uint32))
        check_grads({kk: v.cpu().numpy() for kk, v in grads.items()}, want)
