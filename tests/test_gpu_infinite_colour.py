"""GPU tests that a Gaussian whose colour has overflowed to +inf changes only
the pixels that take it (and, in the backward, only Gaussians that share a
pixel with it): the blends give other pixels weight zero, and zero times
infinity must not reach their sums."""
import numpy as np
import pytest

from paper_2403_01444_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

Y00 = 0.28209479177387814


def scene(colour, seed, n=1500):
    """Small Gaussians; number 0 lies in front of them and has `colour` in channel 0."""
    g = synth.make_gaussians(n, 0, seed)
    g.log_scales -= np.float32(1.2)
    cam_dir = synth.look_at_camera(64, 64).cam_pos / 3.0
    g.means[0] = (cam_dir * 1.2).astype(np.float32) + np.float32([0.03, 0.05, 0.0])
    g.log_scales[0] = -3.6
    g.opacity_logits[0] = 0.5
    g.sh[0, 0, 0] = (colour - 0.5) / Y00 if np.isfinite(colour) else np.inf
    return g


def render(g, width, height, mode, log2):
    from paper_2403_01444_amd import gs3
    cam = synth.look_at_camera(width, height, bg=(0.2, 0.1, 0.3))
    ctx = gs3.Context(g.n, 1 << 20, width, height, sort_mode=mode, grad_record_log2=log2)
    img = ctx.render(gs3.GaussiansGPU.from_host(g), cam).clone()
    _, box, _ = ctx.debug_gaussians(g.n)
    rng = np.random.default_rng(5)
    d = torch.from_numpy(rng.normal(size=(3, height, width)).astype(np.float32)).cuda()
    grads = {"d_uv": ctx.zeros(g.n, 2), "d_conic": ctx.zeros(g.n, 3), "d_opacity": ctx.zeros(g.n),
             "d_rgb": ctx.zeros(g.n, 3)}
    ctx.render_backward(d, grads)
    ctx.check_flags()
    ctx.close()
    return img.cpu().numpy(), box.cpu().numpy(), {k: v.cpu().numpy() for k, v in grads.items()}


# at most 512 tiles (256 with gradient records) take the narrow blends
@pytest.mark.parametrize("width,height", [(90, 70), (400, 352)])
@pytest.mark.parametrize("mode,log2", [("depth_first", 0), ("depth_first", 18), ("radix64", 0)])
def test_infinite_colour_stays_in_its_pixels(width, height, mode, log2):
    plain, box, want = render(scene(1.0, 3), width, height, mode, log2)
    marked, _, _ = render(scene(1e6, 3), width, height, mode, log2)
    img, _, got = render(scene(np.inf, 3), width, height, mode, log2)
    # weights of taken entries are at least 1e-4 / 255: visible against 1e6
    takes = marked[0] != plain[0]
    assert 0 < takes.sum() < 0.2 * takes.size
    assert np.isposinf(img[0][takes]).all()
    assert np.array_equal(img[0][~takes], plain[0][~takes])
    assert np.array_equal(img[1:], plain[1:])
    y, x = np.nonzero(takes)
    apart = (box[:, 0] > x.max()) | (box[:, 2] < x.min()) | (box[:, 1] > y.max()) | (box[:, 3] < y.min())
    near = ~apart & (box[:, 0] <= box[:, 2])
    # among the Gaussians apart, some in tiles of the infinite one
    tiles = (box[:, 0] // 16 <= x.max() // 16) & (box[:, 2] // 16 >= x.min() // 16) & \
            (box[:, 1] // 16 <= y.max() // 16) & (box[:, 3] // 16 >= y.min() // 16)
    assert near.sum() > 0 and (apart & tiles).sum() > 0
    for k in want:
        a, b = got[k][apart], want[k][apart]
        assert np.isfinite(a).all(), k
        if log2:                  # fixed order
            assert np.array_equal(a, b), k
        else:                     # float atomics: see test_gpu_supers.py
            assert np.abs(a - b).max() <= 2e-4 * np.abs(want[k]).max(), k
