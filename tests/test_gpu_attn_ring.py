"""Attention of more than 32 query rows per kv head (attn_ring.hip) at the edges of its row tiles, blocks and splits: alone
(every workgroup finds its one unit itself) and in a crowd that gives every workgroup several units, chains and trees.
Bar: the guards of the other attention tests."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)
from tests.test_gpu_tree import _check_tree_attention

pytestmark = pytest.mark.gpu

CTX = [9, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 2047, 2048, 2049, 4100]     # page, block, turn of a workgroup, split


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("crowd", [0, 1, 250], ids=["alone", "some", "crowd"])
@pytest.mark.parametrize("G,k", [(11, 2), (16, 2), (7, 6), (16, 3), (13, 4), (16, 7)], ids=lambda v: str(v))
def test_many_rows(G, k, crowd, dtype, oracle_mod, pkg):  # noqa: F811
    """33, 48, 49, 64 rows in one group, 65 and 128 in two; requests of every smaller row count beside them."""
    rng = np.random.default_rng(G * 10 + k)
    ctx = [L for L in CTX if L <= (4100 if crowd else 129)] + list(rng.integers(k + 1, 300, crowd))
    spec = [k if i % 3 else i % (k + 1) for i in range(len(ctx))]
    st = W.make_custom_step(G + k, ctx_lens=ctx, spec_lens=spec, n_q_heads=2 * G, n_kv_heads=2, head_dim=128, dtype=dtype,
                            acceptance=False, name=f"ring-{G}-{k}-{crowd}-{dtype}")
    check_attention(st, oracle_mod, pkg)


@pytest.mark.parametrize("G,k,B", [(16, 2, 5), (16, 3, 5), (13, 4, 130), (7, 6, 130)])
def test_many_rows_of_trees(G, k, B, oracle_mod, pkg):  # noqa: F811
    rng = np.random.default_rng(G + k)
    ctx = np.maximum(rng.integers(1, 400, B), k + 1)
    ctx[:5] = [k + 1, 33, 64, 2049, 130]
    st = W.make_custom_step(G * k, ctx_lens=ctx, spec_lens=[k if i % 2 else i % (k + 1) for i in range(B)], n_q_heads=2 * G,
                            n_kv_heads=2, head_dim=128, dtype="bf16", vocab=64, name=f"ring-tree-{G}-{k}")
    W.attach_tree(st, 3)
    _check_tree_attention(st, oracle_mod, pkg)
