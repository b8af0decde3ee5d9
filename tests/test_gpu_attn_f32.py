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


@pytest.mark.parametrize("d,dtype", [(64, "f32"), (128, "f32"), (64, "bf16"), (64, "f16")])
@pytest.mark.parametrize("kind", ["equal and negative", "equal and positive", "far apart"])
@pytest.mark.parametrize("tree", [False, True])
def test_attention_of_very_large_scores(kind, d, dtype, tree, oracle_mod, pkg):  # noqa: F811
    """Scores at the far ends of the storage type (f16: 4e10 in the exponent's units): equal ones average the values, others
    pick the largest, as in the vector kernel and in 64 bits; both these kernels and the head_dim 64 ones."""
    import numpy as np
    from workloads.verify_step import _store, to_f64
    st = W.make_custom_step(77, ctx_lens=[1, 17, 130, 700, 300], spec_lens=[0, 2, 5, 3, 1], n_q_heads=8, n_kv_heads=2, head_dim=d,
                            dtype=dtype, acceptance=False, name=f"large-{dtype}-d{d}")
    big_q, big_k = {"f32": (1e16, 1e16), "bf16": (1e16, 1e16), "f16": (6e4, 6e4)}[dtype]
    if kind == "far apart":
        q, k = to_f64(st.q, dtype), to_f64(st.k_pages, dtype)
        f = {"f32": 1e7, "bf16": 1e7, "f16": 3e3}[dtype]
        q, k = np.clip(q * f, -big_q, big_q), np.clip(k * f, -big_k, big_k)
    else:
        q, k = np.full(st.q.shape, big_q), np.full(st.k_pages.shape, big_k if kind == "equal and positive" else -big_k)
    st.q, st.k_pages = _store(q.astype(np.float32), dtype), _store(k.astype(np.float32), dtype)
    if tree:
        W.attach_tree(st, max_width=2)
        _check_tree_attention(st, oracle_mod, pkg)
    else:
        check_attention(st, oracle_mod, pkg)
