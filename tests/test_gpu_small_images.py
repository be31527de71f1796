"""Images of a few pixels (probes) at the sizes where the split of generation
over wavefronts changes: 2^k pixels and one beside, fewer samples than a
wavefront takes of a pixel and a ragged number more.  Every sample's direction,
pdf, weight and radiance, and the pixels, against the oracle."""
import numpy as np
import pytest

from paper_2607_22780_amd import workloads as W
from test_gpu_render import compare_samples, render_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grt_ctx():
    from paper_2607_22780_amd import grt
    return grt, grt.Context(0)


def probes(npix, seed=0):
    """A 1 x npix strip of valid pixels."""
    gb = W.gbuffer1(24, 24, seed=seed)
    at = np.nonzero(gb.valid)[0][:npix]
    assert len(at) == npix
    return gb.subset(at)


@pytest.mark.parametrize("npix", [1, 2, 3, 5, 16, 17, 31, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("split", [(3, 2, 2), (1, 0, 0), (40, 21, 10)])
def test_small_images(grt_ctx, npix, split):
    grt, ctx = grt_ctx
    s = W.scene1(n=3000, seed=0, s_lo=0.02, s_hi=0.1)
    gpu, ref = render_both(grt, ctx, s, probes(npix), W.envmap(16, 32, seed=1), split, 9)
    edge = compare_samples(gpu["dump"], ref, max_excused=0.01)
    ok = ~edge.any(axis=1)
    assert ok.mean() > 0.5
    np.testing.assert_allclose(gpu["rgb"][ok], ref["rgb"][ok], rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("spp,sizes", [(16, [70, 98304, 98305]), (17, [70, 131072, 131073]), (65, [70, 131073])])
def test_pixel_sums_do_not_depend_on_the_split(grt_ctx, spp, sizes):
    """The same pixels in images on both sides of each line where the split of
    the per-pixel sums changes: sums are in sample order, so equal bit for bit."""
    import torch
    from gpu_util import scene_tensors, t
    grt, ctx = grt_ctx
    base = probes(70)
    scene = grt.Scene(ctx, *scene_tensors(W.scene1(n=3000, seed=0, s_lo=0.02, s_hi=0.1)))
    E = grt.Env(ctx, t(W.envmap(16, 32, seed=1)))
    split = (spp - 8, 5, 3)
    first = None
    for n in sizes:
        G = grt.GBuffer.from_numpy(base.subset(np.arange(n) % 70), torch.device("cuda", 0))
        rgb = grt.render_mis(scene, E, G, split=split, seed=9)["rgb"][:70].cpu().numpy()
        assert np.isfinite(rgb).all() and rgb.any()
        first = rgb if first is None else first
        np.testing.assert_array_equal(rgb.view(np.uint32), first.view(np.uint32), err_msg=str(n))


def test_mesh_frames_do_not_depend_on_the_tiles(grt_ctx):
    """The same pixels relit through the mesh in frames on both sides of the
    number of samples where the query's tiles change, with ragged last tiles."""
    import torch
    from gpu_util import t
    grt, ctx = grt_ctx
    base = W.gbuffer3(24, 24).subset(np.arange(200, 270))
    m = W.mesh3(wall_res=8, segments=12)
    mesh = grt.Mesh(ctx, t(m.verts), t(m.tris))
    at = [t(a) for a in (m.albedo, m.rough, m.metal, m.normal)]
    E = grt.Env(ctx, t(W.envmap(16, 32, seed=1))).prefilter()
    first = None
    for n in (70, 65535, 65536, 65537):
        G = grt.GBuffer.from_numpy(base.subset(np.arange(n) % 70), torch.device("cuda", 0))
        rgb = grt.render_relight_mesh(mesh, E, *at, G, split=(32, 16, 16), seed=4)["rgb"][:70].cpu().numpy()
        assert np.isfinite(rgb).all() and rgb.any()
        first = rgb if first is None else first
        np.testing.assert_array_equal(rgb.view(np.uint32), first.view(np.uint32), err_msg=str(n))
