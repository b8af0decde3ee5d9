"""Attention of more than 32 query rows per kv head over short contexts (attn_rows.hip) at the edges of its row tiles, blocks
and pages and at the widths of the block table up to which it is taken: chains that find their units themselves, chains and
trees by the schedule, in one round and in several. Bar: the guards of the other attention tests."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)
from tests.test_gpu_tree import _check_tree_attention

pytestmark = pytest.mark.gpu


def step(G, k, ctx, dtype, hkv=2, **kw):
    spec = [k if i % 3 else i % (k + 1) for i in range(len(ctx))]
    ctx = [max(L, n + 1) for L, n in zip(ctx, spec)]
    return W.make_custom_step(G + k + len(ctx), ctx_lens=ctx, spec_lens=spec, n_q_heads=hkv * G, n_kv_heads=hkv, head_dim=128, dtype=dtype,
                              name=f"rows-{G}-{k}-{len(ctx)}-{dtype}", **kw)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("longest", [32, 96, 192])
@pytest.mark.parametrize("G,k", [(11, 2), (16, 2), (7, 6), (16, 3), (13, 4), (16, 7)], ids=lambda v: str(v))
def test_short_contexts(G, k, longest, dtype, oracle_mod, pkg):  # noqa: F811
    """33, 48, 49, 64 rows in one group, 65 and 128 in two; 192 tokens: the row split from 49 rows on."""
    ctx = [L for L in (1, 15, 16, 17, 31, 32, 33, 47, 64, 65, 95, 96, 97, 128, 129, 160, 191, 192) if L <= longest]
    check_attention(step(G, k, ctx, dtype, acceptance=False), oracle_mod, pkg)


def test_more_than_the_chip_holds(oracle_mod, pkg):  # noqa: F811
    """Two groups of rows, more possible tokens than direct calls take: units by the schedule, several rounds."""
    ctx = np.random.default_rng(5).integers(1, 177, 800)
    check_attention(step(16, 4, list(ctx), "bf16", hkv=1, acceptance=False), oracle_mod, pkg)


@pytest.mark.parametrize("G,k,B,longest", [(16, 2, 5, 128), (16, 3, 5, 192), (13, 4, 130, 320), (7, 6, 400, 96), (16, 3, 600, 64), (16, 7, 160, 64)])
def test_trees(G, k, B, longest, oracle_mod, pkg):  # noqa: F811
    ctx = np.random.default_rng(G + k + B).integers(1, longest + 1, B)
    ctx[:5] = [k + 1, 33, 32, longest, longest - 1]
    st = step(G, k, list(ctx), "bf16", vocab=64)
    W.attach_tree(st, 3)
    _check_tree_attention(st, oracle_mod, pkg)
