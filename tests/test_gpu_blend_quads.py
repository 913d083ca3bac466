"""GPU tests of the blend's quadrants and blocks: each wave of a tile's
workgroup evaluates only the entries that can reach its 8 x 8 pixels (its
4 x 4, in views of at most 256 tiles), so a scene where
that test could go wrong (thin, tiny, faint and ill-conditioned Gaussians,
ragged images) is compared with every Gaussian evaluated at every pixel of its
box: by the oracle, and from the render's own records."""
import numpy as np
import pytest

from oracle import raster as orc
from paper_2403_01444_amd import synth
from parity import check_grads, check_image

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def scene(kind, n, seed):
    g = synth.make_gaussians(n, 1, seed)
    rng = np.random.default_rng(seed + 1)
    if kind == "thin":            # needles of every direction, aspect up to e^4
        g.log_scales = rng.choice(np.array([-5.5, -4.0, -1.5], np.float32), size=(n, 3)).astype(np.float32)
    elif kind == "tiny":          # below a pixel: the low-pass alone decides the footprint
        g.log_scales -= np.float32(4.0)
        g.opacity_logits += np.float32(3.0)
    elif kind == "faint":         # opacities around and below 1/255
        g.opacity_logits = rng.normal(-5.5, 0.5, n).astype(np.float32)
    elif kind == "long":          # covariances of condition 1e5 and more: the box alone decides
        g.log_scales[:, 0] = 0.5
        g.log_scales[:, 1:] = -7.0
    elif kind == "wall":          # every pixel stops at the last of them, a tile's quadrants at different entries
        cam = synth.look_at_camera(64, 64, azimuth_deg=-9.0)
        zc = cam.world_to_cam[2, :3]
        depth = np.concatenate([np.linspace(2.0, 2.3, 64), rng.uniform(2.5, 3.5, n - 65), [4.0]])
        off = rng.uniform(-1.5, 1.5, (n, 3)) * (np.arange(n) >= 64)[:, None] * (np.arange(n) < n - 1)[:, None]
        off -= (off @ zc)[:, None] * zc
        g.means = (cam.cam_pos + depth[:, None] * zc + off).astype(np.float32)
        big = (np.arange(n) < 64) | (np.arange(n) == n - 1)
        g.log_scales = np.where(big, 3.4, -4.0)[:, None].repeat(3, 1).astype(np.float32)
        p = np.where(big, 0.125, 0.02)
        p[-1] = 0.995
        g.opacity_logits = np.log(p / (1 - p)).astype(np.float32)
    return g


def blend_records(key, box, rec, width, height, bg):
    """Eq. 4 from a render's per-Gaussian records: the exponent in single
    precision in the decision procedure's order, the rest in double.  Returns
    the image, the transmittance and the pixels where a decision (opacity
    1/255, the stop at 1e-4) lies within 1e-5 of its threshold."""
    f = np.float32
    img, T = np.zeros((3, height, width)), np.ones((height, width))
    live, near = np.ones((height, width), bool), np.zeros((height, width), bool)
    order = np.argsort(key, kind="stable")
    for i in order[: int((key != 0xFFFFFFFF).sum())]:
        x0, y0, x1, y1 = box[i]
        u, v, A, B, C, op = rec[i, :6]
        sl = np.s_[y0:y1 + 1, x0:x1 + 1]
        dx, dy = np.arange(x0, x1 + 1).astype(f)[None] - u, np.arange(y0, y1 + 1).astype(f)[:, None] - v
        power = f(-0.5) * ((A * dx) * dx + (C * dy) * dy) - (B * dx) * dy
        raw = float(op) * np.exp(power.astype(np.float64))
        ok = (power <= 0) & (raw >= 1 / 255) & live[sl]
        alpha = np.where(ok, np.minimum(raw, 0.99), 0.0)
        Tn = T[sl] * (1 - alpha)
        near[sl] |= live[sl] & (power <= 0) & (np.abs(raw * 255 - 1) < 1e-5)
        near[sl] |= ok & (np.abs(Tn - 1e-4) < 1e-5 * 1e-4 * 100)
        stop = ok & (Tn < 1e-4)
        live[sl] &= ~stop
        w = np.where(ok & ~stop, alpha * T[sl], 0.0)
        img[(slice(None),) + sl] += w[None] * rec[i, 6:9].astype(np.float64)[:, None, None]
        T[sl] = np.where(ok & ~stop, Tn, T[sl])
    return img + T[None] * np.asarray(bg, np.float64)[:, None, None], T, near


@pytest.mark.parametrize("kind,n,width,height", [("thin", 3000, 97, 61), ("tiny", 4000, 64, 64), ("faint", 1500, 50, 37),
                                                 ("long", 400, 120, 90), ("usual", 1200, 33, 17),
                                                 # past 256 tiles: the 8 x 8 quadrants
                                                 ("thin", 2000, 257, 256), ("tiny", 3000, 300, 290),
                                                 ("faint", 1500, 262, 259), ("long", 300, 272, 257),
                                                 ("usual", 1000, 256, 256), ("usual", 1000, 258, 270),
                                                 # 512 tiles and past them
                                                 ("usual", 1500, 512, 256), ("thin", 2000, 400, 340),
                                                 ("tiny", 3000, 513, 256), ("faint", 1500, 371, 369),
                                                 ("long", 300, 392, 350), ("usual", 1500, 390, 352)])
def test_quadrants_take_every_contributor(kind, n, width, height):
    from paper_2403_01444_amd import gs3
    g = scene(kind, n, n)
    cam = synth.look_at_camera(width, height, azimuth_deg=20.0, bg=(0.3, 0.1, 0.2))
    # "long": single precision cannot project condition 1e5 to the oracle's
    # bar, so only the blend of its records is compared
    projected = kind != "long"
    ref = orc.render(g, cam)
    w = (np.random.default_rng(4).normal(size=(3, height, width)) / (3 * height * width)).astype(np.float32)
    rb = orc.render_backward(g, cam, w.astype(np.float64))
    gg = gs3.GaussiansGPU.from_host(g)
    first = None
    for mode, log2 in (("depth_first", 0), ("depth_first", 16), ("radix64", 0)):
        ctx = gs3.Context(g.n, 1 << 20, width, height, sort_mode=mode, grad_record_log2=log2)
        img = ctx.render(gg, cam).clone()
        T, last = ctx.debug_pixels(cam)
        if projected:
            check_image(img, T, ref, f"{kind} {mode}")
        if first is None:
            key, box, rec = (t.cpu().numpy() for t in ctx.debug_gaussians(g.n))
            want, wantT, near = blend_records(key.view(np.uint32), box, rec, width, height, cam.bg)
            assert near.mean() < 0.05
            # the repository's image bar; a contributor left out shows as up to 1/255
            assert np.abs(img.cpu().numpy() - want)[:, ~near].max() <= 1e-4 * np.abs(want).max()
            assert np.abs(T.cpu().numpy() - wantT)[~near].max() <= 1e-4
            first = (img, T, last)
        else:                     # the same contributors in the same order: bit for bit
            for a, b in zip(first, (img, T, last)):
                assert torch.equal(a, b)
        grads = {"d_means": ctx.zeros(g.n, 3), "d_opacity_logits": ctx.zeros(g.n), "d_rgb": ctx.zeros(g.n, 3)}
        ctx.render_backward(torch.from_numpy(w).cuda(), grads)
        if projected:
            check_grads(grads, rb, f"{kind} {mode}")
        ctx.close()


@pytest.mark.parametrize("log2", [0, 18])
@pytest.mark.parametrize("scene_name,n,width,height", [("surfaces", 6000, 330, 300), ("usual", 3000, 330, 300),
                                                       ("wall", 900, 330, 300), ("thin", 900, 330, 300),
                                                       ("surfaces", 6000, 120, 100), ("wall", 300, 120, 100),
                                                       ("surfaces", 6000, 390, 340), ("usual", 3000, 390, 340),
                                                       ("wall", 1200, 390, 340)])
def test_blends_read_only_what_they_stage(scene_name, n, width, height, log2):
    """The blends do not depend on what earlier kernels left in LDS: with LDS
    full of NaN (the loss of NaN images leaves them there) the image and the
    gradients are the ones without."""
    from paper_2403_01444_amd import gs3
    g = synth.surface_scene(n, 1, 3).gaussians if scene_name == "surfaces" else scene(scene_name, n, 3)
    cam = synth.look_at_camera(width, height, azimuth_deg=-9.0)
    ctx = gs3.Context(g.n, 1 << 20, 1024, 1024, grad_record_log2=log2)
    gg = gs3.GaussiansGPU.from_host(g)
    nan = torch.full((3, 1024, 1024), float("nan"), device="cuda")
    clean = torch.rand((3, 1024, 1024), device="cuda")
    d = torch.from_numpy(np.random.default_rng(2).normal(size=(3, height, width)).astype(np.float32)).cuda()
    out = []
    for image in (clean, nan, nan, nan):
        ctx.loss(image, image)
        img = ctx.render(gg, cam).clone()
        grads = {"d_uv": ctx.zeros(n, 2), "d_conic": ctx.zeros(n, 3), "d_opacity": ctx.zeros(n), "d_rgb": ctx.zeros(n, 3)}
        torch.cuda.synchronize()
        ctx.loss(image, image)
        ctx.render_backward(d, grads)
        out.append((img, grads))
    for img, grads in out[1:]:
        assert torch.equal(img, out[0][0])
        for k, v in grads.items():
            # the sums' order varies (float atomics): see test_gpu_supers.py
            assert float((v - out[0][1][k]).abs().max()) <= 2e-4 * float(out[0][1][k].abs().max()), k
    ctx.close()
