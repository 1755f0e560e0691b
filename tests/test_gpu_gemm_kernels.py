"""Every kernel a prefill GEMM can run on, on the same operands: equal bits, and the float64 result.

The persistent kernel (on all compute units, and on three, where a block walks
full units, halves and a short last row tile) and the seven tile shapes are
named one by one, so nothing here depends on which of them the dispatch would
take.  Rows past M are checked to stay as they were.

Bounds: fp32 sums of K products, in any order, are within S = K 2^-24 sum |a w|
of the exact one; an fp16 output adds half an ulp (2^-11), the hardware's
exponential, reciprocal and the multiplications around them a few fp32 ulps
(2^-20 in all).
"""
import numpy as np
import pytest

from tests import gemm_direct as G
from tests.gpu_common import log, require_gpu

pytestmark = pytest.mark.gpu

PAD = 8   # rows after the last one, to stay untouched
SIZES = [(389, 128), (1300, 384)]   # rows (133 and 20 in the last 256), K


def _operands(torch, M, N, K, fmt):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), generator=gen, device="cuda").half()
    w = (torch.randn((N, K), generator=gen, device="cuda") / K ** 0.5).bfloat16()
    args = dict(M=M, N=N, K=K, A=a, W=G.panels(w.half()) if fmt == "f16" else w, w_f16=int(fmt == "f16"))
    prod = a.double() @ w.double().T.contiguous()
    S = (K * 2.0 ** -24) * (a.double().abs() @ w.double().abs().T.contiguous())
    return gen, args, prod, S


def _check(torch, epi, args, outs, expect):
    """outs: tensors to fill; expect: name -> (rows, columns ...) slice of it, reference, bound."""
    first = None
    for kernel, cus in [(G.PERSISTENT, 256), (G.PERSISTENT, 3)] + [(t, 256) for t in G.TILES]:
        for t in outs.values():
            t.fill_(float("nan"))
        G.run(epi, kernel, cus, **args, **outs)
        torch.cuda.synchronize()
        got = {n: t.clone() for n, t in outs.items()}
        for n, (view, ref, bound) in expect.items():
            x = view(got[n]).double()
            assert x.shape == ref.shape
            err = (x - ref).abs()
            assert bool((err <= bound).all()), (kernel, cus, n, float((err / bound).max()))
            assert int(torch.isnan(got[n]).sum()) == got[n].numel() - ref.numel(), (kernel, cus, n)
        if first is None:
            first = got
        for n in got:
            same = got[n].view(torch.uint8).eq(first[n].view(torch.uint8)).all()
            assert bool(same), f"kernel {kernel} on {cus}: {n} differs from the persistent kernel's"


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("resid", ["resid", "resid_f32"])
def test_residual(M, K, fmt, resid):
    torch = require_gpu()
    N = 768
    log(f"[gemm kernels] residual {M} x {N} x {K} {fmt} {resid}")
    gen, args, prod, S = _operands(torch, M, N, K, fmt)
    x = torch.randn((M, N), generator=gen, device="cuda")
    x = x if resid == "resid_f32" else x.bfloat16()
    ref = x.double() + prod
    out = torch.empty((M + PAD, N), device="cuda")
    bound = S + K * 2.0 ** -24 * x.double().abs() + 2.0 ** -24 * ref.abs()   # the sum starts from the residual
    _check(torch, G.RESID, dict(args, ldo=N, **{resid: x}), dict(out_f32=out), dict(out_f32=(lambda t: t[:M], ref, bound)))


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("resid", ["resid", "resid_f32"])
def test_gated(M, K, fmt, resid):
    torch = require_gpu()
    N = 768
    log(f"[gemm kernels] gated {M} x {N} x {K} {fmt} {resid}")
    gen, args, prod, S = _operands(torch, M, N, K, fmt)
    x = torch.randn((M, N), generator=gen, device="cuda")
    x = x if resid == "resid_f32" else x.bfloat16()
    bias = torch.randn(N, generator=gen, device="cuda").bfloat16()
    gate = torch.randn((3, 2 * N), generator=gen, device="cuda")
    seq = (torch.arange(M, device="cuda") * 3 // M).int()
    g = gate[seq.long(), :N].double()
    ref = x.double() + g * (prod + bias.double())
    out = torch.empty((M + PAD, N), device="cuda")
    bound = g.abs() * (S + 2.0 ** -22 * (prod.abs() + bias.double().abs())) + 2.0 ** -22 * ref.abs()
    _check(torch, G.GATED, dict(args, ldo=N, bias=bias, gate=gate, gate_stride=2 * N, row_seq=seq, **{resid: x}),
           dict(out_f32=out), dict(out_f32=(lambda t: t[:M], ref, bound)))


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_gelu(M, K, fmt):
    torch = require_gpu()
    N = 768
    log(f"[gemm kernels] GELU {M} x {N} x {K} {fmt}")
    gen, args, prod, S = _operands(torch, M, N, K, fmt)
    bias = torch.randn(N, generator=gen, device="cuda").bfloat16()
    z = prod + bias.double()
    ref = 0.5 * z * (1 + torch.tanh((2 / np.pi) ** 0.5 * (z + 0.044715 * z ** 3)))
    out = torch.empty((M + PAD, N), dtype=torch.float16, device="cuda")
    # |gelu'| < 1.13; for z far below zero the exponent is large and its rounding counts: |z| |2u| ulps.
    u = (2 / np.pi) ** 0.5 * (z.abs() + 0.044715 * z.abs() ** 3)
    bound = 1.13 * (S + 2.0 ** -23 * z.abs()) + (2.0 ** -11 + 2.0 ** -20 * (1 + 2 * u)) * ref.abs() + 2.0 ** -24
    _check(torch, G.GELU, dict(args, ldo=N, bias=bias), dict(out=out), dict(out=(lambda t: t[:M], ref, bound)))


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_swiglu(M, K, fmt):
    torch = require_gpu()
    F = 384
    log(f"[gemm kernels] SwiGLU {M} x 2 {F} x {K} {fmt}")
    gen, args, prod, S = _operands(torch, M, 2 * F, K, fmt)
    g, u = prod[:, :F], prod[:, F:]
    act = g * torch.sigmoid(g)
    ref = act * u
    out = torch.empty((M + PAD, F), dtype=torch.float16, device="cuda")
    # |silu'| < 1.1; the exponential's argument is rounded to fp32.
    bound = (1.1 * S[:, :F] * u.abs() + act.abs() * S[:, F:] + (2.0 ** -11 + 2.0 ** -20 * (1 + g.abs())) * ref.abs() +
             2.0 ** -24)
    _check(torch, G.SWIGLU, dict(args, ldo=F, ffn=F), dict(out=out), dict(out=(lambda t: t[:M], ref, bound)))


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("form", ["plain", "bias", "sections", "unrotated"])
@pytest.mark.parametrize("dh", [64, 128])
def test_qkv(M, K, fmt, form, dh):
    torch = require_gpu()
    hq, hkv = (8, 2) if dh == 64 else (4, 1)
    N = (hq + 2 * hkv) * dh
    half = dh // 2
    log(f"[gemm kernels] QKV {M} x {N} x {K} {fmt} head size {dh} {form}")
    gen, args, prod, S = _operands(torch, M, N, K, fmt)
    y = prod
    if form in ("bias", "unrotated"):
        bias = torch.randn(N, generator=gen, device="cuda").bfloat16()
        args["bias"] = bias
        y, S = prod + bias.double(), S + 2.0 ** -23 * (prod.abs() + bias.double().abs())
    y, S = y.reshape(M, -1, dh), S.reshape(M, -1, dh)
    n_pos = 3000
    th = torch.arange(n_pos, device="cuda").double()[:, None] * 1e4 ** (-torch.arange(half, device="cuda") / half).double()
    table = torch.stack([th.cos(), th.sin()], -1).float().contiguous()
    sec = (dh // 8, dh // 8 + 3 * half // 8) if form == "sections" else (half, half)
    pos = torch.randint(0, n_pos, (3 if form == "sections" else 1, M), generator=gen, device="cuda", dtype=torch.int32)
    comp = (torch.arange(half, device="cuda") >= sec[0]).long() + (torch.arange(half, device="cuda") >= sec[1]).long()
    cs = table.double()[pos[comp if form == "sections" else torch.zeros_like(comp)].long().T,
                        torch.arange(half, device="cuda")][:, None]          # [M, 1, half, 2]
    c, s = (cs[..., 0], cs[..., 1]) if form != "unrotated" else (torch.ones_like(cs[..., 0]), torch.zeros_like(cs[..., 0]))
    turn = hq + hkv
    lo, hi, Sl, Sh = y[:, :turn, :half], y[:, :turn, half:], S[:, :turn, :half], S[:, :turn, half:]
    rot = torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
    mag = torch.cat([(lo * c).abs() + (hi * s).abs(), (hi * c).abs() + (lo * s).abs()], -1)
    sum_err = torch.cat([c.abs() * Sl + s.abs() * Sh, c.abs() * Sh + s.abs() * Sl], -1)
    bound = sum_err + 2.0 ** -11 * rot.abs() + 2.0 ** -22 * mag + 2.0 ** -24
    vref, vS = y[:, turn:], S[:, turn:]
    vbound = vS + 2.0 ** -11 * vref.abs() + 2.0 ** -24

    ctx = -(-(M + PAD) // 32) * 32
    row = torch.arange(M, device="cuda")
    q = torch.empty((M + PAD, hq, dh), dtype=torch.float16, device="cuda")
    k = torch.empty((hkv, ctx, dh), dtype=torch.float16, device="cuda")
    v = torch.empty((hkv, ctx // 32, dh, 32), dtype=torch.float16, device="cuda")
    args.update(pos=pos.contiguous(), pos_stride=M if form == "sections" else 0, sec1=sec[0], sec2=sec[1],
                k_off=row * dh, v_off=row // 32 * (32 * dh) + row % 32, kv_head_stride=ctx * dh, hq=hq, hkv=hkv, dh=dh,
                rope=0 if form == "unrotated" else table)
    _check(torch, G.QKV, args, dict(q=q, k=k, v=v), dict(
        q=(lambda t: t[:M], rot[:, :hq], bound[:, :hq]),
        k=(lambda t: t[:, :M].transpose(0, 1), rot[:, hq:], bound[:, hq:]),
        v=(lambda t: t.transpose(2, 3).reshape(hkv, ctx, dh)[:, :M].transpose(0, 1), vref, vbound)))
