"""The rotation of every GEMM's QKV epilogue, bit for bit.

With weights of zero the projection is its bias, so the rotated queries and
keys follow exactly from bf16 values and a given table.  One product of each
output is rounded to fp32 before the fused multiply-add:

* prefill GEMMs: (fma(lo, cos, -(hi sin)), fma(lo, sin, hi cos))
* skinny GEMM:   (fma(lo, cos, -(hi sin)), fma(hi, cos, lo sin))

The other choice differs in the last fp32 bit of half the outputs, which turns
about one fp16 value in 10^4 (a stack of four layers then differs by 1e-4 and
more from one that rounds this way).
"""
import numpy as np
import pytest

from tests import gemm_direct as G
from tests.gpu_common import log, require_gpu

pytestmark = pytest.mark.gpu


def _fma32(a, b, c):
    """fp32 fma: products of an 8-bit and a 24-bit significand fit a long double beside c."""
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(np.float32)


@pytest.mark.parametrize("kernel", [G.SKINNY, G.PERSISTENT, *G.TILES])
@pytest.mark.parametrize("dh", [64, 128])
def test_rotation_bits(dh, kernel):
    torch = require_gpu()
    hq, hkv, K = (30, 1, 128) if dh == 64 else (13, 1, 128)
    heads = hq + 2 * hkv
    if heads * dh % 256:
        hq += 1
        heads += 1
    M = 128 if kernel == G.SKINNY else 2000
    N = heads * dh
    rng = np.random.default_rng(5)
    bias = torch.from_numpy(rng.normal(size=N).astype(np.float32)).to(torch.bfloat16)
    th = rng.uniform(0, 2 * np.pi, (M, dh // 2))
    table = np.stack([np.cos(th), np.sin(th)], -1).astype(np.float32)
    b = bias.to(torch.float32).numpy().reshape(heads, dh)[:hq + hkv]
    lo, hi = b[None, :, :dh // 2], b[None, :, dh // 2:]
    c, s = table[:, None, :, 0], table[:, None, :, 1]
    first = _fma32(lo, c, -(hi * s))
    second = _fma32(hi, c, lo * s) if kernel == G.SKINNY else _fma32(lo, s, hi * c)
    expect = np.concatenate([first, second], -1).astype(np.float16)

    log(f"[rotation] head size {dh}, kernel {kernel}, {M} rows")
    dev = "cuda"
    q = torch.zeros((M, hq, dh), dtype=torch.float16, device=dev)
    k = torch.zeros((hkv, M, dh), dtype=torch.float16, device=dev)
    v = torch.zeros((hkv, -(-M // 32), dh, 32), dtype=torch.float16, device=dev)
    row = torch.arange(M, dtype=torch.int64, device=dev)
    G.run(G.QKV, kernel, A=torch.zeros((M, K), dtype=torch.float16, device=dev),
          W=torch.zeros((N, K), dtype=torch.bfloat16, device=dev), M=M, K=K, N=N, q=q, k=k, v=v,
          pos=row.to(torch.int32), sec1=dh // 2, sec2=dh // 2, k_off=row * dh, v_off=row // 32 * (dh * 32) + row % 32,
          kv_head_stride=v[0].numel(), rope=torch.from_numpy(table).to(dev), bias=bias.to(dev), hq=hq, hkv=hkv, dh=dh)
    torch.cuda.synchronize()
    got = np.concatenate([q.cpu().numpy(), k.cpu().numpy().transpose(1, 0, 2)], 1)
    wrong = int((got.view(np.uint16) != expect.view(np.uint16)).sum())
    log(f"  {wrong} of {expect.size} values differ")
    assert wrong == 0
