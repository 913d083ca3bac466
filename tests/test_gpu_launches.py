"""GPU tests of the paths that replace several launches by one: the
one-workgroup sort, the fused clearing, and the gradient sums that their
reader clears."""
import numpy as np
import pytest

from paper_2403_01444_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 63, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193])
def test_order_around_the_one_workgroup_sort(n):
    """Morton order (30-bit keys, many ties, stable by index) on both sides
    of the size up to which one workgroup sorts."""
    from paper_2403_01444_amd import gs3
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16)
    pts = rng.integers(0, 6, size=(n, 3)).astype(np.float32) / np.float32(8)
    pts[::7] = rng.uniform(0, 1, size=pts[::7].shape).astype(np.float32)
    perm = ctx.morton_order(torch.from_numpy(pts).cuda(), (0, 0, 0), (1, 1, 1)).cpu().numpy()
    q = np.minimum((pts * np.float32(1024)).astype(np.int64), 1023)
    code = np.zeros(n, np.int64)
    for b in range(10):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    assert np.array_equal(perm, np.argsort(code, kind="stable"))
    ctx.close()


@pytest.mark.parametrize("n", [65_537, 262_143, 262_144, 262_145, 524_289, 1_048_577, 2_097_152, 2_097_153])
def test_order_around_the_block_sizes(n):
    """Morton order on both sides of the sizes at which a block takes more
    keys, and past the last of them: whole and ragged last blocks, waves of
    one digit, many ties."""
    from paper_2403_01444_amd import gs3
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16)
    pts = rng.integers(0, 6, size=(n, 3)).astype(np.float32) / np.float32(8)
    pts[n // 3:] = rng.uniform(0, 1, size=pts[n // 3:].shape).astype(np.float32)
    pts[-1] = 0
    perm = ctx.morton_order(torch.from_numpy(pts).cuda(), (0, 0, 0), (1, 1, 1)).cpu().numpy()
    q = np.minimum((pts * np.float32(1024)).astype(np.int64), 1023)
    code = np.zeros(n, np.int64)
    for b in range(10):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + a)
    assert np.array_equal(perm, np.argsort(code, kind="stable"))
    ctx.close()


def test_zero_many_clears_each_array_and_nothing_else():
    from paper_2403_01444_amd import gs3
    ctx = gs3.Context(10, 1 << 10, 16, 16)
    sizes = [1, 3, 4, 1023, 1024, 1025, 0, 4099] + [7] * 12       # more than one launch's worth
    buf = torch.ones(sum(sizes) + 2 * len(sizes) + 8, device="cuda")
    views, at = [], 1                                              # unaligned starts among them
    for s in sizes:
        views.append(buf[at:at + s])
        at += s + 1
    keep = torch.ones_like(buf, dtype=torch.bool)
    at = 1
    for s in sizes:
        keep[at:at + s] = False
        at += s + 1
    ctx.zero(*views)
    assert torch.equal(buf, keep.float())
    ctx.zero()
    ctx.close()


@pytest.mark.parametrize("log2", [0, 6])
def test_backwards_start_from_cleared_sums(log2):
    """A second backward of the same render adds the same gradient again,
    after a render of fewer Gaussians in between and a refused call (log2 6:
    records that overflow into the sums)."""
    from paper_2403_01444_amd import gs3
    g = synth.make_gaussians(3000, 1, 9)
    cam = synth.look_at_camera(80, 60)
    ctx = gs3.Context(g.n, 1 << 18, 80, 60, grad_record_log2=log2)
    gg = gs3.GaussiansGPU.from_host(g)
    few = gs3.GaussiansGPU.from_host(g.subset(np.arange(500)))
    d = torch.from_numpy(np.random.default_rng(1).normal(size=(3, 60, 80)).astype(np.float32)).cuda()
    one = {"d_uv": ctx.zeros(g.n, 2), "d_rgb": ctx.zeros(g.n, 3)}
    ctx.render(gg, cam)
    with pytest.raises(gs3.GS3Error):
        ctx.render_backward(d, {"d_uv": ctx.zeros(g.n, 2), "vspace_grad": ctx.zeros(g.n)})
    ctx.render_backward(d, one)
    ctx.render(few, cam)
    ctx.render_backward(d, {"d_uv": ctx.zeros(500, 2)})
    two = {k: v.clone() for k, v in one.items()}
    ctx.render(gg, cam)
    ctx.render_backward(d, two)
    for k in one:
        # twice the sum; each run's float atomics add a Gaussian's few tiles in another order
        assert float((two[k] - 2 * one[k]).abs().max()) <= 1e-5 * float(one[k].abs().max())
    ctx.close()


@pytest.mark.parametrize("n,rows,rf", [(1, 3, 1), (257, 300, 3), (1000, 1700, 4), (333, 333, 12), (129, 200, 27),
                                       (700, 1000, 48), (5, 9, 1000)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gathered_rows(n, rows, rf, shift):
    """Rows by index, four floats at a time where rows and arrays allow it
    (shift: arrays that start one float past an aligned address)."""
    from paper_2403_01444_amd import gs3
    rng = np.random.default_rng(n)
    ctx = gs3.Context(max(n, rows), 1 << 10, 16, 16)
    src = torch.rand(rows * rf + 1, device="cuda")[shift:shift + rows * rf].view(rows, rf)
    dst = torch.full((n * rf + 2,), -1.0, device="cuda")
    perm = torch.from_numpy(rng.integers(0, rows, n).astype(np.int32)).cuda()
    gs3.gs3_gather_rows(ctx.h, src, perm, n, rf, dst[shift:shift + n * rf])
    assert torch.equal(dst[shift:shift + n * rf].view(n, rf), src[perm.long()])
    assert float(dst[shift + n * rf]) == -1.0
    ctx.close()
