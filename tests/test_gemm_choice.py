"""Which kernels the GPU tests' prefill calls reach, by the library's own rule (host only).

A new fit of the rule's constants moves the calls to other kernels without a
word: this fails when an epilogue no longer meets the persistent kernel or
loses the variety of tile shapes that the GPU tests claim.
"""
import os

import pytest

from paper_2608_01785_amd import workloads as W
from tests import gemm_direct as G
from tests import test_gpu_gemm_tiles as tiles
from tests import test_gpu_mrope as mrope

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_01785_amd", "libhorizon.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libhorizon.so not built")


def products(s):
    """(epilogue, N, K) of a layer's or block's four projections."""
    if isinstance(s, W.DitShape):
        return [("qkv", 3 * s.hidden, s.hidden), ("gated", s.hidden, s.hidden), ("gelu", s.mlp, s.hidden),
                ("gated", s.hidden, s.mlp)]
    qd = s.n_q_heads * s.head_dim
    return [("qkv", (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim, s.hidden), ("resid", s.hidden, qd),
            ("swiglu", 2 * s.ffn, s.hidden), ("resid", s.hidden, s.ffn)]


def reached(cases):
    seen = {}
    for s, rows, budgets in cases:
        for epi, n, k in products(s):
            seen.setdefault(epi, set()).update(G.choice(rows, n, k, b) for b in budgets)
    return seen


def test_every_epilogue_meets_the_persistent_kernel_and_four_tile_shapes():
    seen = reached([({"talker": W.TALKER, "tiny": W.TINY}[n], rows, tiles.BUDGETS) for n, rows, _ in tiles.LAYER_CASES] +
                   [(W.DIT, rows, tiles.DIT_BUDGETS) for rows, _ in tiles.DIT_CASES])
    assert set(seen) == {"qkv", "resid", "swiglu", "gelu", "gated"}
    for epi, kernels in seen.items():
        assert G.PERSISTENT in kernels and len(kernels) >= 5, (epi, kernels)


def test_each_format_of_the_gated_product_meets_the_persistent_kernel():
    for fmt in ("f16", "bf16"):
        kernels = reached([(W.DIT, rows, tiles.DIT_BUDGETS) for rows, f in tiles.DIT_CASES if f == fmt])
        assert G.PERSISTENT in kernels["gated"], fmt


def test_sectioned_rotation_meets_both_kernels():
    epi, n, k = products(W.TALKER)[0]
    assert G.choice(mrope.PERSISTENT_ROWS, n, k, 64) == G.PERSISTENT
    assert G.choice(mrope.PERSISTENT_ROWS, n, k, 128) in G.TILES


@pytest.mark.parametrize("shape", [W.THINKER, W.THINKER_MIXED, W.TALKER, W.TINY, W.DIT], ids=lambda s: str(s.hidden))
def test_choice_is_defined_everywhere(shape):
    for _, n, k in products(shape):
        for rows in (1, 2, 63, 64, 65, 127, 129, 255, 256, 257, 1000, 4096, 9151, 65536):
            for cus in (1, 3, 64, 200, 256):
                assert G.choice(rows, n, k, cus) in (G.PERSISTENT, *G.TILES)
