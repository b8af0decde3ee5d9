"""The two metadata kernels of scheduled attention calls: up to 256 requests with up to 8192 possible splits take the one
that keeps everything on chip. A block table wide enough for more splits sends the same call to the general one; who
computes what differs, results do not."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.test_gpu_parity import pkg  # noqa: F401  (fixture)
from tests.test_gpu_tree import _check_tree_attention

pytestmark = pytest.mark.gpu

ITEMS = 8192            # possible splits up to which the lengths of all of them fit on chip
SPLIT = 2048            # of calls with 256 (request, kv head) pairs and more


@pytest.mark.parametrize("tree", [False, True], ids=["chain", "tree"])
@pytest.mark.parametrize("B,hq,hkv,d,k,dtype", [(256, 8, 8, 128, 3, torch.bfloat16), (255, 12, 6, 64, 2, torch.float16),
                                                (64, 28, 4, 128, 5, torch.bfloat16), (65, 32, 8, 128, 6, torch.float16),
                                                (33, 32, 16, 64, 1, torch.float32), (40, 64, 8, 128, 10, torch.bfloat16)],
                         ids=lambda v: str(v).replace("torch.", ""))
def test_both_metadata_kernels_give_the_same(B, hq, hkv, d, k, dtype, tree, pkg):  # noqa: F811
    rng = np.random.default_rng(B + hq)
    ctx = np.maximum(rng.integers(1, 300, B), k + 1)
    ctx[[0, 1, 2, 3, B // 2, B - 2, B - 1]] = [SPLIT, SPLIT + 1, k + 1, 2 * SPLIT + 1, 21000, 5 * SPLIT, 4095]
    spec = rng.integers(0, k + 1, B)
    spec[[0, 3, B - 1]] = k
    pages = -(-ctx // 16)
    ids = rng.permutation(int(pages.sum())).astype(np.int32)
    starts = np.concatenate([[0], np.cumsum(pages)])
    narrow = np.full((B, int(pages.max())), -1, np.int32)
    for i in range(B):
        narrow[i, :pages[i]] = ids[starts[i]:starts[i + 1]]
    wide = np.full((B, (ITEMS // B + 1) * (SPLIT // 16)), -1, np.int32)
    wide[:, :narrow.shape[1]] = narrow
    assert B * -(-wide.shape[1] * 16 // SPLIT) > ITEMS >= B * -(-narrow.shape[1] * 16 // SPLIT)
    gen = torch.Generator(device="cuda").manual_seed(B)
    TQ = int(spec.sum()) + B
    q = torch.randn((TQ, hq, d), generator=gen, device="cuda").to(dtype)
    kp, vp = (torch.randn((len(ids), hkv, 16, d), generator=gen, device="cuda").to(dtype) for _ in range(2))
    parents = np.concatenate([[-1] + [int(rng.integers(0, j)) for j in range(1, n + 1)] for n in spec]).astype(np.int32)
    dev = lambda a: torch.tensor(np.asarray(a, np.int32), device="cuda")  # noqa: E731
    kw = dict(parents=dev(parents)) if tree else {}
    outs = [pkg.verify_attn(q, kp, vp, dev(t), dev(ctx), dev(spec), max_spec_len=k, **kw) for t in (narrow, wide)]
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(*outs)


@pytest.mark.parametrize("hq,hkv,d,k,dtype", [(8, 8, 64, 2, "f32"), (16, 8, 64, 3, "bf16"), (8, 8, 128, 3, "f16"), (32, 8, 128, 6, "bf16"),
                                              (64, 8, 128, 4, "bf16")], ids=lambda v: str(v))
@pytest.mark.parametrize("B,longest", [(66, 900), (80, 300)])
def test_some_compute_units_take_a_third_unit(B, longest, hq, hkv, d, k, dtype, pkg, oracle_mod):  # noqa: F811
    """A few more units than a round of two per compute unit holds; kernels and metadata have to agree on who takes which."""
    ctx = longest // 3 + (longest - longest // 3) * np.random.default_rng(B).permutation(B) // B
    st = W.make_custom_step(B + k, ctx_lens=ctx, spec_lens=[k - i % 2 for i in range(B)], n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                            vocab=64, name=f"thirds-{B}-{hq}-{d}-{dtype}")
    W.attach_tree(st, 2)
    _check_tree_attention(st, oracle_mod, pkg)
