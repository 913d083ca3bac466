"""GPU tests that the NTC's paths give the same gradient where a rule on sizes
chooses between them: prepared lists against the table gradient of means that
were not prepared (parts of the table summed in LDS, global atomics for large
tables), at and past the number of points processed at a time."""
import numpy as np
import pytest

from paper_2403_01444_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


@pytest.mark.parametrize("n,log2_T,precision", [
    (1025, 15, "f32"),          # a slice of two rows of points
    (30_000, 10, "f16"),        # every level one part, ragged
    (70_001, 16, "bf16"),       # 8192-entry parts: more than half of the most
    (3000, 18, "f32"),          # global atomics against counted lists of several parts a level
    (3000, 19, "f32"),          # more parts than the points are read for: global atomics, sorted lists
    (262_144 + 65, 15, "f16"),  # a second round of points
])
def test_unprepared_gradient_matches_the_prepared(n, log2_T, precision):
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig(log2_T=log2_T)
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16, ntc=cfg, precision=precision)
    p = synth.ntc_init_params(cfg, 1)
    p[: cfg.num_table_params()] *= 1000.0
    ctx.ntc_load(p)
    m = cuda(rng.uniform(-1.25, 1.25, size=(n, 3)))
    gm, gq = cuda(rng.normal(size=(n, 3)) * 1e-3), cuda(rng.normal(size=(n, 4)) * 1e-3)
    tok = ctx.ntc_prepare(m)
    ctx.ntc_backward(m, gm, gq, tok)
    a = ctx.ntc_grads().double()
    ctx.ntc_zero_grads()
    ctx.ntc_backward(m, gm, gq)
    b = ctx.ntc_grads().double()
    # Both add the same float32 products.  An entry's m addends summed in
    # float32 are within m 2^-24 of their absolute sum A; the fullest entries
    # (level 0: 8 n / 4913 addends, a few hundred, of either sign, A up to 20
    # times the largest sum) stay below 5e-4 of the largest entry.  Rounds of
    # points scale the half-precision activations batch by batch, alike.
    t = cfg.num_table_params()
    assert float((a[:t] - b[:t]).abs().max()) <= 5e-4 * float(a[:t].abs().max())
    assert float((a[t:] - b[t:]).abs().max()) <= 5e-4 * float(a[t:].abs().max())
    assert float(a[:t].abs().max()) > 0
    ctx.close()


@pytest.mark.parametrize("n", [1, 255, 257, 4099])
def test_prepared_lists_repeat(n):
    """The contribution lists and their order depend on the means alone: two
    contexts that prepare the same means give the same gradient bit for bit,
    whatever was prepared before."""
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig()
    rng = np.random.default_rng(n)
    pts = rng.uniform(-1.2, 1.2, size=(n, 3)).astype(np.float32)
    pts[: n // 2] = pts[0]                       # one cell: every lane on the same entries
    m, other = cuda(pts), cuda(rng.uniform(-1, 1, size=(5000, 3)))
    gm, gq = cuda(rng.normal(size=(n, 3)) * 1e-3), cuda(rng.normal(size=(n, 4)) * 1e-3)
    out = []
    for first in (False, True):
        ctx = gs3.Context(5000, 1 << 10, 16, 16, ntc=cfg, precision="f32")
        p = synth.ntc_init_params(cfg, 1)
        p[: cfg.num_table_params()] *= 1000.0
        ctx.ntc_load(p)
        if first:
            ctx.ntc_prepare(other)
        tok = ctx.ntc_prepare(m)
        for _ in range(2):
            ctx.ntc_zero_grads()
            ctx.ntc_backward(m, gm, gq, tok)
            out.append(ctx.ntc_grads()[: cfg.num_table_params()].clone())
        ctx.close()
    assert all(torch.equal(out[0], o) for o in out[1:])
    assert float(out[0].abs().max()) > 0


@pytest.mark.parametrize("n,log2_T,precision", [
    (16_384, 15, "f16"), (16_385, 15, "bf16"), (17_407, 10, "f16"),
    (20_000, 16, "f16"),          # levels that do not fit: encoded in the MLP's launch
    (524_288 + 77, 15, "bf16"),   # a second round of points
])
def test_encoding_apart_is_the_same(n, log2_T, precision):
    """Many points are encoded in a launch of their own, few in the MLP's: the
    same bits either way, for points on and past the box's faces too, and a
    backward takes the kept encoding of either as it would compute it."""
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig(log2_T=log2_T)
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16, ntc=cfg, precision=precision)
    p = synth.ntc_init_params(cfg, 1)
    p[: cfg.num_table_params()] *= 1000.0
    ctx.ntc_load(p)
    x = rng.uniform(-1.25, 1.25, size=(n, 3)).astype(np.float32)
    x[:3] = [[1.2, -1.2, 0.0], [1.2, 1.2, 1.2], [-1.2, -1.2, -1.2]]
    x[3:6] = [[np.nan, 0, 0], [np.inf, 0, 0], [0, -np.inf, 0]]
    x[-1] = [0.3, 1.2, -0.4]
    m = cuda(x)
    piece = 8000
    parts = [ctx.ntc_forward(m[k:k + piece].contiguous()) for k in range(0, n, piece)]
    dmu, dq = ctx.ntc_forward(m)
    assert torch.equal(dmu, torch.cat([a for a, _ in parts])) and torch.equal(dq, torch.cat([b for _, b in parts]))
    gm, gq = cuda(rng.normal(size=(n, 3)) * 1e-3), cuda(rng.normal(size=(n, 4)) * 1e-3)
    tok = ctx.ntc_prepare(m)
    grads = []
    for forward in (False, True):
        if forward:
            got = ctx.ntc_forward(m, token=tok)
            assert torch.equal(got[0], dmu) and torch.equal(got[1], dq)
        ctx.ntc_zero_grads()
        ctx.ntc_backward(m, gm, gq, tok)
        grads.append(ctx.ntc_grads())
    t = cfg.num_table_params()
    assert torch.equal(grads[0][:t], grads[1][:t])
    # the weights' partial sums meet in float atomics: at most 16 of them in any order
    assert float((grads[0][t:] - grads[1][t:]).abs().max()) <= 16 * 2 ** -24 * 16 * float(grads[0][t:].abs().max())
    ctx.close()


@pytest.mark.parametrize("n,log2_T,spread", [(1, 15, 1.25), (17, 15, 1.25), (2000, 15, 1.25), (3000, 15, 0.01),
                                             (100, 10, 1.25), (6000, 16, 0.3)])
def test_few_points_gather(n, log2_T, spread):
    """The gather of few points (a lane an entry, longer lists 16 lanes) gives
    the table gradient of the scattered one, and the same bits each time."""
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig(log2_T=log2_T)
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16, ntc=cfg)
    p = synth.ntc_init_params(cfg, 1)
    p[: cfg.num_table_params()] *= 1000.0
    ctx.ntc_load(p)
    m = cuda(rng.uniform(-spread, spread, size=(n, 3)))
    gm, gq = cuda(rng.normal(size=(n, 3)) * 1e-3), cuda(rng.normal(size=(n, 4)) * 1e-3)
    tok = ctx.ntc_prepare(m)
    t = cfg.num_table_params()
    got = []
    for token in (tok, tok, 0):
        ctx.ntc_zero_grads()
        ctx.ntc_backward(m, gm, gq, token)
        got.append(ctx.ntc_grads()[:t].double())
    assert torch.equal(got[0], got[1])
    # the same float32 products in another order: an entry's up to 8 n addends
    # (all points in a cell or two) differ by their number times 2^-24 of their
    # absolute sum, a walk of either sign that stays below the bound of the
    # tests above by far
    scale = float(got[0].abs().max())
    assert float((got[0] - got[2]).abs().max()) <= 5e-4 * scale
    ctx.close()


@pytest.mark.parametrize("n,kind", [(220_000, "box"), (323_584, "box"), (323_585, "box"), (220_001, "cell"),
                                    (230_000, "corner"), (260_003, "out")])
def test_lists_by_slices(n, kind):
    """The lists of many points, kept slice by slice: the table gradient of the
    scattered one, and the same bits each time.  cell: an entry's list reaches
    over lanes, rounds and waves; corner: most entries have none; out: slices
    without a contribution."""
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig()
    rng = np.random.default_rng(n)
    x = rng.uniform(-1.25, 1.25, size=(n, 3))
    if kind == "cell":
        x = 0.01 + 0.0005 * rng.uniform(size=(n, 3))
    elif kind == "corner":
        x = -1.2 + 0.3 * rng.uniform(size=(n, 3))
    elif kind == "out":
        x[30_000:90_000] = 2.0
        x[-70_000:] = -3.0
    m = cuda(x)
    gm, gq = cuda(rng.normal(size=(n, 3)) * 1e-3), cuda(rng.normal(size=(n, 4)) * 1e-3)
    t = cfg.num_table_params()
    p = synth.ntc_init_params(cfg, 1)
    p[:t] *= 1000.0
    got = []
    for again in range(2):
        ctx = gs3.Context(n, 1 << 10, 16, 16, ntc=cfg, precision="f16")
        ctx.ntc_load(p)
        if again:
            ctx.ntc_prepare(cuda(rng.uniform(-1, 1, size=(n // 2, 3))))   # other lists before
        tok = ctx.ntc_prepare(m)
        ctx.ntc_backward(m, gm, gq, tok)
        got.append(ctx.ntc_grads()[:t])
        if again:
            ctx.ntc_backward(m, gm, gq, tok)       # adds to what is there
            twice = ctx.ntc_grads()[:t]
            ctx.ntc_zero_grads()
            ctx.ntc_backward(m, gm, gq)
            got.append(ctx.ntc_grads()[:t])
        ctx.close()
    assert torch.equal(got[0], got[1]) and torch.equal(twice, got[0] + got[1])
    # float32 sums of the same products against sums in double of 8192 points
    # and less: the fullest entry adds up to 8 n products ("cell"), of random
    # sign, in runs of a few hundred, so 1000 roundings of 2^-24 relative to
    # sums that are as large as the result within a factor of a few
    a, b = got[0].double(), got[2].double()
    assert float(a.abs().max()) > 0
    assert float((a - b).abs().max()) <= 5e-4 * float(a.abs().max())
