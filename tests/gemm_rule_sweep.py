"""Times every prefill GEMM kernel over the products of the layers and blocks: the evidence for the rule that chooses
between them (not a test; needs a GPU):

    python -m tests.gemm_rule_sweep OUT.csv

One line per product, weight format, row count and budget, with the product's own epilogue, on the budget's CU-masked
stream: microseconds of the persistent kernel and of the seven tile shapes, and the rule's choice.  A summary follows
on the standard output.
"""
import sys

import numpy as np

from tests import gemm_direct as G

ROWS = (130, 200, 280, 389, 520, 700, 1000, 1400, 2048, 3073, 4500, 6500, 9151)
BUDGETS = (64, 96, 128, 160, 192, 256)
# name, epilogue, N, K, (query heads, key/value heads, head size), row limit
PRODUCTS = [
    ("thinker qkv", G.QKV, 4608, 3584, (28, 4, 128), 1 << 20), ("thinker o", G.RESID, 3584, 3584, None, 1 << 20),
    ("thinker gate/up", G.SWIGLU, 37888, 3584, None, 1 << 20), ("thinker down", G.RESID, 3584, 18944, None, 1 << 20),
    ("talker qkv", G.QKV, 3072, 1024, (16, 16, 64), 5000), ("talker o", G.RESID, 1024, 1024, None, 5000),
    ("talker gate/up", G.SWIGLU, 8192, 1024, None, 5000), ("talker down", G.RESID, 1024, 4096, None, 5000),
    ("dit o", G.GATED, 1024, 1024, None, 5000), ("dit fc1", G.GELU, 4096, 1024, None, 5000),
    ("dit fc2", G.GATED, 1024, 4096, None, 5000),
]


def operands(torch, epi, M, N, K, heads, fmt, copies):
    gen = torch.Generator(device="cuda").manual_seed(1)
    args = dict(M=M, N=N, K=K, A=torch.randn((M, K), generator=gen, device="cuda").half(), w_f16=int(fmt == "f16"))
    w = (torch.randn((N, K), generator=gen, device="cuda") / K ** 0.5)
    w = G.panels(w.half()) if fmt == "f16" else w.bfloat16()
    weights = [w] + [w.clone() for _ in range(copies - 1)]
    if epi == G.RESID or epi == G.GATED:
        args.update(out_f32=torch.empty((M, N), device="cuda"), resid_f32=torch.randn((M, N), generator=gen, device="cuda"),
                    ldo=N)
    if epi == G.GATED or epi == G.GELU:
        args.update(bias=torch.zeros(N, dtype=torch.bfloat16, device="cuda"), ldo=N)
    if epi == G.GATED:
        args.update(gate=torch.randn((4, 6 * N), generator=gen, device="cuda"), gate_stride=6 * N,
                    row_seq=(torch.arange(M, device="cuda") * 4 // M).int())
    if epi == G.GELU:
        args.update(out=torch.empty((M, N), dtype=torch.float16, device="cuda"))
    if epi == G.SWIGLU:
        args.update(out=torch.empty((M, N // 2), dtype=torch.float16, device="cuda"), ldo=N // 2, ffn=N // 2)
    if epi == G.QKV:
        hq, hkv, dh = heads
        ctx, row = -(-M // 32) * 32, torch.arange(M, device="cuda")
        half = torch.float16
        args.update(q=torch.empty((M, hq, dh), dtype=half, device="cuda"), k=torch.empty((hkv, ctx, dh), dtype=half, device="cuda"),
                    v=torch.empty((hkv, ctx // 32, dh, 32), dtype=half, device="cuda"), pos=row.int(), sec1=dh // 2,
                    sec2=dh // 2, k_off=row * dh, v_off=row // 32 * (32 * dh) + row % 32, kv_head_stride=ctx * dh, hq=hq,
                    hkv=hkv, dh=dh, rope=torch.randn((M, dh // 2, 2), generator=gen, device="cuda"))
    return args, weights


def main(path):
    import torch
    from paper_2608_01785_amd import binding
    ctx = binding.Context(0, budgets=BUDGETS)
    rows = []
    with open(path, "w") as f:
        f.write("product,format,M,N,K,cus,persistent," + ",".join(f"tile{t}" for t in G.TILES) + ",choice\n")
        for name, epi, N, K, heads, limit in PRODUCTS:
            for fmt in ("f16", "bf16"):
                for M in [m for m in ROWS if m <= limit]:
                    args, weights = operands(torch, epi, M, N, K, heads, fmt, 4)
                    torch.cuda.synchronize()
                    for cus in BUDGETS:
                        h = binding.hs_context_stream(ctx, cus, binding.HS_ROLE_SHARED)
                        s = torch.cuda.ExternalStream(h)
                        t = []
                        for kernel in (G.PERSISTENT, *G.TILES):
                            n, us = 4, []
                            launches = [G.call(epi, kernel, cus, stream=h, W=w, **args) for w in weights]
                            for rep in range(4):
                                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                                e[0].record(s)
                                for i in range(n):
                                    launches[i % len(launches)]()
                                e[1].record(s)
                                torch.cuda.synchronize()
                                if rep:
                                    us.append(e[0].elapsed_time(e[1]) * 1e3 / n)
                                else:
                                    n = int(min(40, max(4, 2.0 / max(e[0].elapsed_time(e[1]) / n, 1e-3))))
                            t.append(min(us))
                        c = G.choice(M, N, K, cus)
                        rows.append((name, fmt, M, cus, t, c))
                        f.write(f"{name},{fmt},{M},{N},{K},{cus}," + ",".join(f"{x:.1f}" for x in t) + f",{c}\n")
                    del args, weights, launches
                print(name, fmt, flush=True)
    for fmt in ("f16", "bf16"):
        sel = [r for r in rows if r[1] == fmt]
        best = np.array([min(r[4]) for r in sel])
        pick = np.array([r[4][r[5] + 1] for r in sel])
        pers = np.array([r[4][0] for r in sel])
        print(f"{fmt}: {len(sel)} launches; the choice takes {np.mean(pick / best) - 1:.1%} more than the fastest kernel "
              f"on average, {np.max(pick / best) - 1:.1%} at most; against the persistent kernel {np.max(pick / pers) - 1:.1%} "
              f"at most, {np.sum(pick) / np.sum(pers):.2f} of its time in all, {np.exp(np.mean(np.log(pick / pers))):.2f} "
              f"in the geometric mean")
        for i in np.argsort(-(pick / best))[:12]:
            r = sel[i]
            print(f"  {r[0]} M={r[2]} on {r[3]}: choice {r[5]} {pick[i]:.1f}, best {int(np.argmin(r[4])) - 1} {best[i]:.1f}, "
                  f"persistent {pers[i]:.1f}")
    ctx.close()


if __name__ == "__main__":
    main(sys.argv[1])
