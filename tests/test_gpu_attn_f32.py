"""Matrix-core attention for fp32, head_dim 64 and 128 (csrc/attn_f32.hip), and the calls without a metadata kernel,
against the CPU oracle: row-tile counts 1, 2, 4 and more than one row group, contexts around the 16-token page, the
64-token turn of a workgroup and the split length, small batches (direct) and batches with a schedule, chains and trees.

Tolerance: fp32 products and sums over head_dim and up to a few thousand tokens of N(0, 1) values; the fp32 guard of the
other attention tests (2e-5)."""
import pytest

import workloads as W
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)
from tests.test_gpu_tree import _check_tree_attention

pytestmark = pytest.mark.gpu

SHAPES = [
    # ctx_lens, spec_lens, Hq, Hkv
    ([1, 2, 16, 17, 63, 64, 65], [0, 1, 0, 2, 1, 3, 0], 2, 2),                 # direct, one row tile
    ([130, 127, 129, 640], [8, 0, 7, 3], 8, 2),                                # direct, three row tiles used of four
    ([1030], [5], 32, 8),                                                      # one request, two row tiles, many splits
    ([90, 700, 33], [10, 12, 0], 16, 2),                                       # G = 8: 104 rows, two row groups
    ([128] * 40 + [2500] * 3, [1] * 40 + [4] * 3, 16, 8),                      # schedule, two splits
    ([5, 300] * 130, [2, 0] * 130, 4, 2),                                      # more requests than a direct call takes
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"B{len(s[0])}-L{max(s[0])}-k{max(s[1])}-{s[2]}x{s[3]}")
def test_attention_f32_edges(shape, d, oracle_mod, pkg):  # noqa: F811
    ctx, spec, hq, hkv = shape
    st = W.make_custom_step(320, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="f32",
                            acceptance=False, name=f"f32-d{d}")
    check_attention(st, oracle_mod, pkg)


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (4, 2, 128)])
def test_tree_attention_f32_edges(hq, hkv, d, oracle_mod, pkg):  # noqa: F811
    ctx = [1, 64, 65, 40, 300, 2100, 33, 16, 700, 17]
    spec = [0, 63, 63, 39, 7, 30, 32, 15, 1, 5]
    st = W.make_custom_step(321, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="f32",
                            acceptance=False, name=f"f32-tree-d{d}")
    W.attach_tree(st, max_width=4)
    _check_tree_attention(st, oracle_mod, pkg)
