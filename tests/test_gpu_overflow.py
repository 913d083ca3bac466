"""More pairs than the capacity, far enough past it that the places kept for a
view run out: the room of the tile lists (views of few tiles) and the blocks of
walked entries (larger views).  A CPU test computes from the oracle's
projection that the scenes do that; the GPU tests check that the render stays
in bounds, reports the overflow, and that the tiles with a place are whole."""
import numpy as np
import pytest

from oracle import raster as orc
from paper_2403_01444_amd import synth

torch = pytest.importorskip("torch")

BLOCK = 256            # entries of a walked block
SCENES = {             # n, width, height, capacity in pairs
    "few tiles": (4000, 64, 64, 2000),
    "many tiles": (20_000, 400, 352, 20_000),
}


def scene(name):
    """Gaussians over the whole view: 2% visible, the others below the opacity
    threshold, so that every pixel walks its whole list."""
    n, width, height, cap = SCENES[name]
    g = synth.make_gaussians(n, 0, n)
    g.log_scales[:] = 1.0
    p = np.where(np.random.default_rng(n).random(n) < 0.02, 0.02, 0.003)
    g.opacity_logits = np.log(p / (1 - p)).astype(np.float32)
    return g, synth.look_at_camera(width, height, bg=(0.3, 0.2, 0.1)), cap


def kept_entries(g, cam, cap):
    """Tiles x entries that the supers' lists, cut at cap, hold for each tile,
    and the Gaussians in depth order."""
    p = orc.preprocess(g, cam)
    order = np.argsort(p["key"], kind="stable")
    order = order[p["visible"][order] > 0]
    x0, y0, x1, y1 = p["rect"][order].T
    tx, ty = (cam.width + 15) // 16, (cam.height + 15) // 16
    count, used = np.zeros((ty, tx), np.int64), 0
    for sy in range(0, ty, 4):
        for sx in range(0, tx, 4):
            meets = np.nonzero((x0 <= sx + 3) & (x1 >= sx) & (y0 <= sy + 3) & (y1 >= sy))[0][: max(cap - used, 0)]
            used += meets.size
            for y in range(sy, min(sy + 4, ty)):
                for x in range(sx, min(sx + 4, tx)):
                    count[y, x] = ((x0[meets] <= x) & (x1[meets] >= x) & (y0[meets] <= y) & (y1[meets] >= y)).sum()
    return count, order


def test_scenes_run_out_of_room():
    g, cam, cap = scene("few tiles")
    count, _ = kept_entries(g, cam, cap)
    assert count.size <= 512 and (count == cap).all()
    assert count.sum() > 5 * (cap // BLOCK + count.size) * BLOCK
    g, cam, cap = scene("many tiles")
    count, _ = kept_entries(g, cam, cap)
    assert count.size > 512 and (count[:4, :4] == cap).all() and count.sum() == 16 * cap
    needed = -(-count // BLOCK) - 1          # past each tile's own block
    assert needed.clip(0).sum() > 10 * (cap // BLOCK)


def both(name):
    """The render with the scene's capacity and one with room for every pair."""
    from paper_2403_01444_amd import gs3
    g, cam, cap = scene(name)
    gg = gs3.GaussiansGPU.from_host(g)
    d = torch.from_numpy(np.random.default_rng(1).normal(size=(3, cam.height, cam.width)).astype(np.float32)).cuda()
    out = []
    for pairs in (cap, 1 << 24):
        ctx = gs3.Context(g.n, pairs, cam.width, cam.height)
        img = ctx.render(gg, cam).clone()
        grads = {"d_uv": ctx.zeros(g.n, 2), "d_rgb": ctx.zeros(g.n, 3), "d_opacity": ctx.zeros(g.n)}
        ctx.render_backward(d, grads)
        walked = ctx.debug_sums()[1]
        _, last = ctx.debug_pixels(cam)
        torch.cuda.synchronize()
        if pairs == cap:
            assert ctx.debug_counts()[1] == 1
            with pytest.raises(gs3.GS3Error) as e:
                ctx.check_flags()
            assert e.value.status == gs3.GS3_ECAPACITY
        else:
            ctx.check_flags()
        ctx.close()
        assert all(bool(torch.isfinite(t).all()) for t in grads.values())
        out.append((img.cpu().numpy(), walked, last.cpu().numpy()))
    return out


@pytest.mark.gpu
def test_tile_lists_past_their_room():
    from paper_2403_01444_amd import gs3
    g, cam, cap = scene("few tiles")
    count, order = kept_entries(g, cam, cap)
    (img, _, last), _ = both("few tiles")
    # what a tile whose list has its place shows: the first cap Gaussians
    first = g.subset(order[:cap])
    ctx = gs3.Context(cap, 1 << 20, cam.width, cam.height)
    want = ctx.render(gs3.GaussiansGPU.from_host(first), cam).cpu().numpy()
    ctx.check_flags()
    ctx.close()
    bg = np.asarray(cam.bg, np.float32)[:, None, None]
    whole = empty = 0
    for y in range(0, 64, 16):
        for x in range(0, 64, 16):
            t = np.s_[:, y:y + 16, x:x + 16]
            whole += np.array_equal(img[t], want[t])
            empty += bool((img[t] == bg).all())
    slots = (cap // BLOCK + count.size) * BLOCK
    # one more is cut, perhaps past its last contributor
    assert whole in (slots // cap, slots // cap + 1) and empty >= 16 - slots // cap - 1
    assert last.max() <= cap


@pytest.mark.gpu
def test_walked_blocks_past_their_room():
    (img, walked, last), (want, _, want_last) = both("many tiles")
    # the first super's lists fill the capacity; its tiles are whole, with a place for what they walked or not
    assert np.array_equal(img[:, :64, :64], want[:, :64, :64])
    assert np.array_equal(last[:64, :64], want_last[:64, :64]) and want_last[:64, :64].min() > 10_000
    rest = np.ones(img.shape[1:], bool)
    rest[:64, :64] = False
    assert (img[:, rest] == np.asarray((0.3, 0.2, 0.1), np.float32)[:, None]).all() and not last[rest].any()
    # tiles without a place for their last contributor are left out by the backward
    longest = [int(last[y:y + 16, x:x + 16].max()) for y in range(0, 64, 16) for x in range(0, 64, 16)]
    assert walked < sum(longest)
