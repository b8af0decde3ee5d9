"""Matrix-core attention for head_dim 64 (csrc/attn_d64.hip) against the CPU oracle: row-tile counts 1, 2, 4 and more
than one row group, contexts around the 16-token page, the 64-token block, the 256-token turn of a workgroup and the
split length, chains and trees.

Tolerance on the fp32 accumulator: scores and sums in fp32 over head_dim 64 products of N(0, 1) values; the weights
carry 24 (bf16) or 22 (f16) bits, so both types are held to the fp32 guard of the other attention tests (2e-5)."""
import pytest

import workloads as W
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)
from tests.test_gpu_tree import _check_tree_attention

pytestmark = pytest.mark.gpu

SHAPES = [
    # ctx_lens, spec_lens, Hq, Hkv
    ([1, 2, 16, 17, 63, 64, 65], [0, 1, 0, 2, 1, 3, 0], 2, 2),                 # one row tile, partly filled
    ([255, 256, 257, 319, 321], [8, 0, 7, 3, 8], 8, 2),                        # three row tiles used of four
    ([511, 513, 2047, 2049, 4097], [3, 1, 0, 3, 2], 8, 2),                     # splits of this few pairs: 256 tokens
    ([40, 300, 1500], [5, 0, 8], 56, 8),                                       # G = 7: 63 rows, the last one alone in none
    ([90, 700, 33], [10, 12, 0], 16, 2),                                       # G = 8: 104 rows, two row groups
    ([128] * 40 + [2500] * 3, [1] * 40 + [4] * 3, 32, 8),                      # more units than workgroups of a round share
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"B{len(s[0])}-L{max(s[0])}-k{max(s[1])}-{s[2]}x{s[3]}")
def test_attention_d64_edges(shape, dtype, oracle_mod, pkg):  # noqa: F811
    ctx, spec, hq, hkv = shape
    st = W.make_custom_step(640, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=64, dtype=dtype,
                            acceptance=False, name=f"d64-{dtype}")
    check_attention(st, oracle_mod, pkg, tol=2e-5)


@pytest.mark.parametrize("dtype,hq,hkv", [("bf16", 2, 2), ("f16", 8, 2)])
def test_tree_attention_d64_edges(dtype, hq, hkv, oracle_mod, pkg):  # noqa: F811
    ctx = [1, 64, 65, 40, 300, 2100, 33, 16, 700, 17]
    spec = [0, 63, 63, 39, 7, 30, 32, 15, 1, 5]
    st = W.make_custom_step(641, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=64, dtype=dtype,
                            acceptance=False, name=f"d64-tree-{dtype}")
    W.attach_tree(st, max_width=4)
    _check_tree_attention(st, oracle_mod, pkg)
