"""The clock record of a GEMM launch covers the whole launch, whichever kernel runs it."""
import pytest

from tests import gemm_direct as G
from tests.gpu_common import log, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", [G.PERSISTENT, *G.TILES])
def test_record_covers_the_launch(kernel):
    torch = require_gpu()
    M, N, K = 4096, 8192, 1024   # a dozen rounds and more of the smallest tiles
    gen = torch.Generator(device="cuda").manual_seed(1)
    a = torch.randn((M, K), generator=gen, device="cuda").half()
    w = torch.randn((N, K), generator=gen, device="cuda").half().reshape(K // 32, N, 32)
    x = torch.randn((M, N), generator=gen, device="cuda")
    out = torch.empty((M, N), device="cuda")
    rec = torch.zeros((4, 4), dtype=torch.int64, device="cuda")
    args = dict(M=M, K=K, N=N, A=a, W=w, w_f16=1, out_f32=out, resid_f32=x, ldo=N)
    G.run(G.RESID, kernel, **args)
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    e[0].record()
    for i in range(4):
        G.run(G.RESID, kernel, clock=rec[i], **args)
    e[1].record()
    torch.cuda.synchronize()
    us = e[0].elapsed_time(e[1]) * 1e3 / 4
    c0, w0, c1, w1 = rec.double().cpu().unbind(1)
    ticks_us, mhz = (w1 - w0) / 100.0, (c1 - c0) / (w1 - w0) * 100.0   # 100 MHz constant clock
    log(f"[clock] kernel {kernel}: launch {us:.0f} us, recorded {ticks_us.tolist()} us, {mhz.tolist()} MHz")
    assert bool((ticks_us > 0.5 * us).all())           # events bracket launches and the gaps between them
    assert bool(((mhz > 300) & (mhz < 2600)).all())    # the card runs at up to 2400 MHz


def test_read_clock():
    torch = require_gpu()
    from paper_2608_01785_amd import binding, workloads as W
    from paper_2608_01785_amd.device_data import to_device, upload_weights
    from tests.gpu_common import workspace
    shape, rows = W.TALKER, 385
    ctx = binding.Context(0, budgets=(64, 128))
    try:
        w = upload_weights(W.make_weights(shape, 1, 3))
        x = to_device(W.token_rows(4, rows, shape.hidden))
        y = torch.empty(x.shape, dtype=torch.float32, device="cuda")
        ws = workspace(torch, shape, rows, 1, rows)
        torch.cuda.synchronize()
        binding.hs_timing_enable(ctx, True)
        kinds = set()
        for cus in (64, 128):   # the gate/up product runs persistent on 64 CUs and in tiles on 128
            kinds.add(G.choice(rows, 2 * shape.ffn, shape.hidden, cus) == G.PERSISTENT)
            binding.hs_shared_stage_forward(ctx, shape, w, x, y, [0, rows], cu_budget=cus, workspace=ws)
        for kind in ("qkv", "o_proj", "gate_up", "down"):
            mhz, n = binding.hs_timing_read_clock(ctx, kind)
            log(f"[clock] {kind}: {mhz:.0f} MHz over {n} launches")
            assert n == 2 and 300 < mhz < 2600
        binding.hs_timing_enable(ctx, False)
        assert kinds == {True, False}
    finally:
        torch.cuda.synchronize()
        ctx.close()
