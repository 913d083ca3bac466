"""GPU tests of the binning where a Gaussian meets many supers: scenes whose
rectangles fill the view, views cut into parts of rows of supers, and both
kinds of scatter in one render, against the 64-bit sort of every pair; and what
such a scene's binning may cost."""
import numpy as np
import pytest

from paper_2403_01444_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def view_filling(n, seed, offset=2.0):
    g = synth.make_gaussians(n, 0, seed)
    g.log_scales += np.float32(offset)
    g.opacity_logits -= np.float32(3.0)
    return g


def lists(g, cam, pairs, mode):
    from paper_2403_01444_amd import gs3
    ctx = gs3.Context(g.n, pairs, cam.width, cam.height, sort_mode=mode)
    img = ctx.render(gs3.GaussiansGPU.from_host(g), cam).clone()
    keys, vals = ctx.debug_pairs()
    ctx.check_flags()
    ctx.close()
    return img, keys, vals


# (n, width, height, offset): offset None for half view-filling, half tiny
CASES = [
    (600, 1024, 512, 2.0),        # 16 x 8 supers, eight parts; every super dense
    (513, 4096, 640, 2.5),        # 64 columns; a chunk of one Gaussian
    (1500, 1100, 500, None),      # dense and sparse supers in the same chunks
    (520, 40, 20000, 2.0),        # one column of 313 supers: parts of 64 rows
    (40_000, 64, 64, 0.0),        # one super
    (270_000, 130, 70, -1.0),     # more than 512 chunks: one part
]


@pytest.mark.parametrize("n,width,height,offset", CASES)
def test_dense_lists_match_the_sorted_pairs(n, width, height, offset):
    g = view_filling(n, n, 2.0 if offset is None else offset)
    if offset is None:
        g.log_scales[::2] = -5.5
    cam = synth.look_at_camera(width, height, azimuth_deg=11.0, bg=(0.1, 0.2, 0.3))
    if height > 4 * width:
        cam.fx = cam.fy = 0.29 * height
    a, b = (lists(g, cam, 1 << 24, mode) for mode in ("depth_first", "radix64"))
    assert a[1].numel() > n // 2
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_binning_of_view_filling_gaussians_costs_less_than_their_blend():
    """20,000 Gaussians over most of 1920 x 1080: the scatter is a fraction of
    the forward blend (an eighth when this was written; ten times the blend when
    it walked the rectangles once per 6144 entries of a chunk)."""
    from paper_2403_01444_amd import gs3
    g = synth.make_gaussians(20_000, 1, 1)
    g.log_scales += np.float32(2.0)
    cam = synth.look_at_camera(1920, 1080, azimuth_deg=11.0)
    ctx = gs3.Context(g.n, 200_000_000, 1920, 1080)
    gg = gs3.GaussiansGPU.from_host(g)
    img = ctx.render(gg, cam)
    ctx.check_flags()
    gs3.gs3_profile_enable(ctx.h, True)
    gs3.gs3_profile_reset(ctx.h)
    for _ in range(5):
        ctx.render(gg, cam, image=img)
    scatter, _ = gs3.gs3_profile_query(ctx.h, "bin_scatter")
    blend, _ = gs3.gs3_profile_query(ctx.h, "blend_fwd")
    assert 0 < scatter < blend
    ctx.close()
