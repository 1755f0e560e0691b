"""Decode steps at the edges of the single-row attention's tiles and ranges, in a cache full of NaN.

Rows whose keys end one before, at and one past the edges of a 32-key tile, of
a round of four waves' tiles and of a key range (1024 keys for head size 64,
512 for 128).  Every position that no row attends to holds NaN, in the pages of
a paged cache too: a missing mask shows, also on values whose weight is zero.
"""
import numpy as np
import pytest

from oracle import layer as ref
from paper_2608_01785_amd import workloads as W
from tests.gpu_common import TOL, err_ratio, log, require_gpu
from tests.util import f64, h64, weights_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    from paper_2608_01785_amd import binding
    ctx = binding.Context(0, budgets=(128,))
    yield torch, ctx
    torch.cuda.synchronize()
    ctx.close()


# Cached rows; the step's own key comes on top.
EDGES = [0, 1, 30, 31, 32, 62, 63, 64, 126, 127, 128, 255, 256, 510, 511, 512, 1022, 1023, 1024, 1535, 2047, 2048]


@pytest.mark.parametrize("page", [0, 64, 256], ids=lambda p: f"page{p}")
@pytest.mark.parametrize("shape", [W.TALKER, W.THINKER_MIXED], ids=["64", "128"])
def test_decode_step_at_tile_edges(env, shape, page):
    torch, ctx = env
    from paper_2608_01785_amd import binding
    from paper_2608_01785_amd.device_data import DeviceCache, PagedCache, to_device, upload_weights
    kv_lens = np.array(EDGES, np.int32)
    batch, top = len(EDGES), -(-(max(EDGES) + 1) // 256) * 256
    layers = W.make_weights(shape, 1, 61)
    x = W.token_rows(62, batch, shape.hidden)
    prefix = W.make_cache(shape, 1, kv_lens, seed=63)
    log(f"[decode edges] head size {shape.head_dim}, page {page}")
    expect, _ = ref.decode_step(f64(x), weights_f64(layers), shape, kv_lens, [[h64(k) for k in prefix.k[0]]],
                                [[h64(v) for v in prefix.v[0]]])
    dims = dict(n_kv_heads=shape.n_kv_heads, head_dim=shape.head_dim, fill=float("nan"))
    if page:
        per = top // page
        table = np.random.default_rng(64).permutation(batch * per).reshape(batch, per)
        cache = PagedCache(1, batch * per, page, table=table, **dims)
    else:
        cache = DeviceCache(1, batch, top, **dims)
    for b in range(batch):
        cache.load_prefix(0, b, prefix.k[0][b], prefix.v[0][b])
    ws = torch.empty(binding.hs_workspace_size_paged(shape, batch, batch, top, page), dtype=torch.uint8, device="cuda")
    wdev, xd = upload_weights(layers), to_device(x)
    y = torch.full(xd.shape, float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    binding.hs_downstream_decode_step(ctx, shape, wdev, xd, y, cache.as_arg(), kv_lens, 128, None, ws)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    for b in range(batch):
        assert np.isfinite(got[b]).all(), f"{kv_lens[b]} cached rows"
    e = err_ratio(got, expect)
    log(f"  max err / rms = {e:.3e}")
    assert e <= TOL
