"""GPU tests of calls of one context on several streams without ordering
between them: an NTC forward without a token writes its outputs and no
workspace, so it may run beside others and beside a backward."""
import numpy as np
import pytest

from paper_2403_01444_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n", [16_384, 120_001])
def test_forwards_overlap(precision, n):
    from paper_2403_01444_amd import gs3
    cfg = synth.NTCConfig()
    rng = np.random.default_rng(n)
    ctx = gs3.Context(n, 1 << 10, 16, 16, ntc=cfg, precision=precision)
    p = synth.ntc_init_params(cfg, 1)
    p[: cfg.num_table_params()] *= 1000.0
    ctx.ntc_load(p)
    means = [torch.from_numpy(rng.uniform(-1, 1, size=(n, 3)).astype(np.float32)).cuda() for _ in range(3)]
    gm = torch.from_numpy((rng.normal(size=(n, 3)) * 1e-3).astype(np.float32)).cuda()
    gq = torch.from_numpy((rng.normal(size=(n, 4)) * 1e-3).astype(np.float32)).cuda()
    want = [[t.clone() for t in ctx.ntc_forward(m)] for m in means]
    ctx.ntc_backward(means[2], gm, gq)
    grad = ctx.ntc_grads()
    ctx.ntc_zero_grads()
    outs = [[(ctx.empty(n, 3), ctx.empty(n, 4)) for _ in range(8)] for _ in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for k in range(8):
        for s in (0, 1):
            gs3.gs3_set_stream(ctx.h, streams[s].cuda_stream)
            ctx.ntc_forward(means[s], *outs[s][k])
        if k == 3:
            gs3.gs3_set_stream(ctx.h, streams[2].cuda_stream)
            ctx.ntc_backward(means[2], gm, gq)
    torch.cuda.synchronize()
    ctx.use_current_stream()
    for s in (0, 1):
        for dmu, dq in outs[s]:
            assert torch.equal(dmu, want[s][0]) and torch.equal(dq, want[s][1])
    # float atomics in another order: see test_gpu_ntc_paths.py
    assert float((ctx.ntc_grads() - grad).abs().max()) <= 5e-4 * float(grad.abs().max())
    ctx.close()
