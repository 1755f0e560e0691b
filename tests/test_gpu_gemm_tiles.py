"""Prefill layers and denoising steps against the reference and, bit for bit, across budgets.

Each budget sends a layer's four projections to kernels of its own choice, so
equal outputs at every budget compare whole calls whose kernels differ; one of
them is compared with the float64 reference.  Which kernels the cases reach is
pinned on the CPU in test_gemm_choice.py: every epilogue meets the persistent
kernel and at least four tile shapes, not all seven (test_gpu_gemm_kernels.py
names each kernel for each epilogue).  Row counts sit at the edges of 64-, 96-,
128-, 160- and 192-row tiles and past the 256-row tiles' first sizes.
"""
import numpy as np
import pytest

from oracle import dit as dit_ref
from oracle import layer as ref
from paper_2608_01785_amd import workloads as W
from tests.gpu_common import TOL, err_ratio, log, require_gpu, workspace
from tests.util import f64, weights_f64

pytestmark = pytest.mark.gpu

BUDGETS = (64, 96, 128, 160, 192, 256)


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    from paper_2608_01785_amd import binding
    ctx = binding.Context(0, budgets=BUDGETS)
    yield torch, ctx
    torch.cuda.synchronize()
    ctx.close()


LAYER_CASES = [
    ("talker", 129, "f16"), ("talker", 193, "bf16"), ("talker", 257, "f16"), ("talker", 385, "bf16"),
    ("talker", 641, "f16"), ("talker", 1100, "bf16"), ("talker", 3330, "f16"), ("tiny", 191, "f16"),
    ("tiny", 2305, "bf16"),
]


@pytest.mark.parametrize("shape_name,rows,fmt", LAYER_CASES)
def test_layer_tiles(env, shape_name, rows, fmt):
    torch, ctx = env
    from paper_2608_01785_amd import binding
    from paper_2608_01785_amd.device_data import prepare_f16, to_device, upload_weights
    shape = {"talker": W.TALKER, "tiny": W.TINY}[shape_name]
    layers = W.make_weights(shape, 1, 71, qkv_bias_std=0.1)
    off = [0, rows // 3, rows]
    x = W.token_rows(72, rows, shape.hidden)
    expect, _ = ref.stack_forward(f64(x), weights_f64(layers), shape, off)
    wdev = upload_weights(layers)
    if fmt == "f16":
        wdev = prepare_f16(ctx, wdev)
    ws = workspace(torch, shape, rows, 2, rows)
    first = None
    for b in BUDGETS:
        log(f"[{shape_name} {rows} rows {fmt}] {b} CUs")
        y = torch.full((rows, shape.hidden), float("nan"), dtype=torch.float32, device="cuda")
        xd = to_device(x)
        torch.cuda.synchronize()
        binding.hs_shared_stage_forward(ctx, shape, wdev, xd, y, off, cu_budget=b, workspace=ws)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        if first is None:
            first = got
            e = err_ratio(got, expect)
            log(f"  max err / rms = {e:.3e}")
            assert e <= TOL
        np.testing.assert_array_equal(got, first)


DIT_BUDGETS = (64, 96, 160, 192)   # the complements of 192, 160, 96 and 64
DIT_CASES = [(65, "f16"), (161, "bf16"), (449, "f16"), (800, "bf16"), (1025, "bf16"), (3073, "f16"), (3329, "bf16")]


@pytest.mark.parametrize("rows,fmt", DIT_CASES)
def test_dit_tiles(env, rows, fmt):
    torch, ctx = env
    from paper_2608_01785_amd import binding
    from paper_2608_01785_amd.device_data import prepare_dit_f16, to_device, upload_weights
    shape = W.DIT
    layers = W.make_dit_weights(shape, 1, 81)
    off = [0, rows // 4, rows]
    x = W.token_rows(82, rows, shape.hidden)
    cond = W.dit_cond(83, 2, shape.hidden)
    expect = dit_ref.dit_forward(f64(x), cond.astype(np.float64), weights_f64(layers), shape, off)
    wdev = upload_weights(layers)
    if fmt == "f16":
        wdev = prepare_dit_f16(ctx, wdev)
    ws = torch.empty(binding.hs_dit_workspace_size(shape, rows, 2), dtype=torch.uint8, device="cuda")
    first = None
    for b in DIT_BUDGETS:
        log(f"[dit {rows} rows {fmt}] {b} CUs")
        y = torch.full((rows, shape.hidden), float("nan"), dtype=torch.float32, device="cuda")
        xd, cd = to_device(x), torch.from_numpy(cond).to("cuda")
        torch.cuda.synchronize()
        binding.hs_dit_forward(ctx, shape, wdev, xd, y, cd, off, b, None, ws)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        if first is None:
            first = got
            e = err_ratio(got, expect)
            log(f"  max err / rms = {e:.3e}")
            assert e <= TOL
        np.testing.assert_array_equal(got, first)
