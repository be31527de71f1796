"""Environment tables where the kernels' chunks and strides change: rows and
columns around a chunk of the running sums, black rows, maps narrower and wider
than a block's step.  Sampling tables bit for bit, prefiltered ones to the
relighting tests' bar."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


@pytest.mark.parametrize("H,W", [(1, 1), (2, 7), (3, 255), (5, 257), (1, 1023), (2, 1024), (1, 1025), (1, 2049),
                                 (1027, 3), (17, 300)])
def test_env_tables(grt_ctx, H, W):
    grt, ctx = grt_ctx
    from gpu_util import t
    g = np.random.default_rng([H, W])
    rgb = np.exp(g.normal(-1.0, 1.5, (H, W, 3))).astype(np.float32)
    if H > 1:
        rgb[H // 2] = 0.0  # a row with no light: uniform steps
    E = grt.Env(ctx, t(rgb)).prefilter()
    torch.cuda.synchronize()
    marg, cond = (a.cpu().numpy() for a in E.tables())
    wm, wc = O.env_cdf(rgb)
    np.testing.assert_array_equal(marg, wm.reshape(marg.shape))
    np.testing.assert_array_equal(cond, wc.reshape(cond.shape))
    for got, want in zip(E.relight_tables()[:2], O.env_prefilter(rgb)):
        np.testing.assert_allclose(got.cpu().numpy(), want.reshape(got.shape), rtol=1e-6, atol=1e-7)
