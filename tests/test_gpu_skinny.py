"""The skinny GEMM at the edges of its two loops (fragments for a short K, whole lines for a long one): stages per wave
from none to seven, odd last pairs, either side of the line between the loops, K splits of unequal length, row counts
at the edges of the 32-row subtiles, one and two weight subtiles, both weight formats and activation layouts.

The reference is the float64 product of the same fp16 and bf16 values.  fp32
sums of K products, in any order, stay within K * 2^-24 * sum |a w| of it (half
an ulp a step), to which the residual's addition adds one more rounding.
"""
import numpy as np
import pytest

from tests import gemm_direct as G
from tests.gpu_common import log, require_gpu

pytestmark = pytest.mark.gpu


def _run(torch, M, K, N, fmt, k8, splits, resident=0):
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    a = torch.randn((M, K), generator=gen, device="cuda").half()
    w = (torch.randn((N, K), generator=gen, device="cuda") * 0.05).bfloat16()
    x = torch.randn((M, N), generator=gen, device="cuda")
    out = torch.full((M, N), float("nan"), device="cuda")
    args = dict(M=M, K=K, N=N, W=w, A=a, out_f32=out, resid_f32=x, ldo=N, w_resident=resident)
    if fmt == "f16":
        args.update(W=G.panels(w.half()), w_f16=1)
    if k8:
        rows = 32 if M <= 32 else 64 if M <= 64 else 128
        pad = torch.full((K // 8, rows, 8), float("nan"), dtype=torch.float16, device="cuda")
        pad[:, :M] = a.reshape(M, K // 8, 8).transpose(0, 1)
        args.update(A=pad, k8_rows=rows)
    if splits:
        strips, subtiles = N // 32, 1 if M <= 32 else 2 if M <= 64 else 4
        args.update(part=torch.empty(strips * splits * subtiles * 1024, device="cuda"),
                    counters=torch.zeros(strips, dtype=torch.int32, device="cuda"))
    log(f"[skinny] {M} x {N} x {K} {fmt} k8={k8} splits={splits} resident={resident}")
    for _ in range(2):   # the second finds the counters as the first left them
        out.fill_(float("nan"))
        G.run(G.RESID, G.SKINNY, **args)
        torch.cuda.synchronize()
        prod = a.double() @ w.double().T.contiguous()
        bound = (K * 2.0 ** -24) * (a.double().abs() @ w.double().abs().T.contiguous()) + 2.0 ** -23 * x.double().abs()
        err = (out.double() - (prod + x.double())).abs()
        log(f"  largest share of the bound {float((err / bound).max()):.3f}")
        assert bool((err <= bound).all())


@pytest.mark.parametrize("fmt,k8,resident", [("f16", True, 0), ("f16", False, 1), ("bf16", False, 0)])
@pytest.mark.parametrize("M", [1, 33, 128])
@pytest.mark.parametrize("K", [128, 256, 384, 512, 640, 768, 896, 1024, 1152, 1536, 1664])
def test_stage_counts(M, K, fmt, k8, resident):
    _run(require_gpu(), M, K, 256, fmt, k8, 0, resident)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M,K", [(1, 256), (32, 512), (1, 768), (1, 896), (33, 512), (64, 640), (33, 1536), (64, 1664),
                                 (65, 768), (128, 896), (65, 1536), (128, 1664)])
def test_gate_up(M, K, fmt):
    """Two weight subtiles per block.  |silu'| < 1.1; an fp16 output adds half an ulp (2^-11), the exponential and the
    reciprocal a few fp32 ulps (2^-20 with the rounding of the argument)."""
    torch = require_gpu()
    F = 256
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    a = torch.randn((M, K), generator=gen, device="cuda").half()
    w = (torch.randn((2 * F, K), generator=gen, device="cuda") / K ** 0.5).bfloat16()
    out = torch.full((M, F), float("nan"), dtype=torch.float16, device="cuda")
    log(f"[skinny gate/up] {M} x 2 {F} x {K} {fmt}")
    G.run(G.SWIGLU, G.SKINNY, M=M, K=K, N=2 * F, A=a, W=G.panels(w.half()) if fmt == "f16" else w, w_f16=int(fmt == "f16"),
          out=out, ldo=F, ffn=F)
    torch.cuda.synchronize()
    prod = a.double() @ w.double().T.contiguous()
    S = (K * 2.0 ** -24) * (a.double().abs() @ w.double().abs().T.contiguous())
    g, u = prod[:, :F], prod[:, F:]
    act = g * torch.sigmoid(g)
    ref = act * u
    bound = (1.1 * S[:, :F] * u.abs() + act.abs() * S[:, F:] + (2.0 ** -11 + 2.0 ** -20 * (1 + g.abs())) * ref.abs() +
             2.0 ** -24)
    assert bool(((out.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("M,K,splits", [(32, 2048, 4), (31, 2176, 4), (64, 2560, 5), (65, 4224, 8)])
def test_splits(M, K, splits):
    _run(require_gpu(), M, K, 256, "f16", True, splits)
