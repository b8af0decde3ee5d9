"""Attention calls with and without a metadata kernel, at the same edges: small batches find their units themselves
(direct), the same requests among more than 256 others go through the schedule. Contexts around the page, the block, the
turn of a workgroup and the shortest splits; one, two and more row tiles; enough splits for every form of the combine
kernel. Bar: the guards of the other attention tests."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # ctx_lens, spec_lens, Hq, Hkv
    ([1, 2, 16, 17, 31, 32, 33], [0, 1, 0, 2, 1, 3, 0], 4, 4),                 # one block and less
    ([127, 128, 129, 511, 513], [3, 0, 7, 3, 8], 8, 2),                        # splits of 128 tokens, up to 36 rows
    ([1500], [5], 32, 8),                                                      # 12 splits: four wavefronts per row combine
    ([9000, 40], [3, 0], 16, 2),                                               # many splits beside a single one
    ([700, 90], [10, 7], 64, 8),                                               # 88 rows: two row groups
    ([4097, 4096, 4095], [0, 1, 2], 8, 1),
]


@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (128, "f16"), (64, "bf16"), (64, "f32"), (128, "f32")])
@pytest.mark.parametrize("crowd", [0, 260], ids=["direct", "scheduled"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"B{len(s[0])}-L{max(s[0])}-k{max(s[1])}-{s[2]}x{s[3]}")
def test_attention_direct_and_scheduled(shape, crowd, d, dtype, oracle_mod, pkg):  # noqa: F811
    ctx, spec, hq, hkv = shape
    rng = np.random.default_rng(crowd + d)
    more = rng.integers(1, 40, crowd)
    at = crowd // 2
    st = W.make_custom_step(128 + d, ctx_lens=[*more[:at], *ctx, *more[at:]], spec_lens=[*[0] * at, *spec, *[0] * (crowd - at)],
                            n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype, acceptance=False, name=f"direct-{crowd}-{dtype}")
    check_attention(st, oracle_mod, pkg)


@pytest.mark.parametrize("B,top,hq,hkv,d,dtype", [(300, 40, 32, 8, 128, "bf16"),     # 2400 units, no combine
                                                  (70, 512, 8, 8, 64, "f16"), (70, 528, 8, 8, 64, "f16"),
                                                  (60, 1008, 32, 8, 128, "bf16"), (60, 1040, 32, 8, 128, "bf16"),
                                                  (90, 30, 64, 8, 128, "bf16"), (90, 300, 64, 8, 128, "bf16"),
                                                  (40, 300, 32, 8, 128, "f32"), (100, 512, 16, 8, 64, "f32")])
def test_attention_short_contexts_around_the_rule(B, top, hq, hkv, d, dtype, oracle_mod, pkg):  # noqa: F811
    rng = np.random.default_rng(B + top)
    spec = rng.integers(0, 6 if hq == 64 else 4, B)
    ctx = np.maximum(rng.integers(1, top + 1, B), spec + 1)
    ctx[B // 2] = top
    st = W.make_custom_step(B + top, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                            acceptance=False, name=f"short-{B}-{top}")
    check_attention(st, oracle_mod, pkg)


def test_attention_direct_with_a_wide_block_table(oracle_mod, pkg):  # noqa: F811
    """A block table far wider than the contexts: most possible splits do not exist, and the entries behind a request's
    pages are not page ids."""
    import torch
    from tests.harness import compare_attention, to_device
    st = W.make_custom_step(5, ctx_lens=[300, 33], spec_lens=[2, 1], n_q_heads=8, n_kv_heads=2, head_dim=128, dtype="bf16",
                            acceptance=False)
    dev = to_device(st, acceptance=False)
    ref, _ = oracle_mod.verify_attn(st.q, st.k_pages, st.v_pages, st.block_table, st.ctx_lens, st.spec_lens, dtype=st.dtype)
    wide = torch.full((2, 1024), -1, dtype=torch.int32, device="cuda")
    wide[:, :dev.block_table.shape[1]] = dev.block_table
    for plan in ("run", "reuse"):                      # a direct call needs no metadata in the workspace
        ws = torch.full((64 << 20,), 255, dtype=torch.uint8, device="cuda")
        out = pkg.verify_attn(dev.q, dev.k_pages, dev.v_pages, wide, dev.ctx_lens, dev.spec_lens, max_spec_len=2, out_dtype=0,
                              workspace=ws, plan=plan)
        torch.cuda.synchronize()
        assert compare_attention(out, ref, None, "bf16")["max_abs_vs_f64"] <= 2e-5


@pytest.mark.parametrize("B,lo,hi,hq,hkv,k", [(62, 2500, 2600, 64, 8, 4), (70, 2500, 2600, 64, 8, 4), (40, 3000, 3600, 64, 8, 8),
                                              (76, 1, 8193, 64, 8, 4), (1100, 1, 50, 16, 1, 2), (140, 1, 4600, 28, 4, 7)])
def test_attention_long_splits_around_the_rule(B, lo, hi, hq, hkv, k, oracle_mod, pkg):  # noqa: F811
    """Row-split kernel: many long requests, one and two row groups, contexts at the edges of one and two splits of 2048 tokens,
    more requests than threads of the plan kernel."""
    rng = np.random.default_rng(B + k)
    spec = rng.integers(0, k + 1, B)
    spec[0] = k
    ctx = np.maximum(rng.integers(lo, hi + 1, B), spec + 1)
    ctx[np.arange(6) * (B // 8) + 1] = [2047, 2048, 2049, min(hi, 4096), min(hi, 4097), max(hi, 2050)]
    st = W.make_custom_step(B + k, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, dtype="bf16",
                            acceptance=False, name=f"long-{B}-{k}")
    check_attention(st, oracle_mod, pkg)


@pytest.mark.parametrize("hq,k", [(64, 4), (64, 8), (32, 4)])
def test_attention_of_a_request_does_not_depend_on_the_lengths_of_the_others(hq, k, pkg):  # noqa: F811
    """How a request is cut into splits follows from its own length and the dims of the call, so the same request among
    long and among short ones gives the same bits (all requests read one sequence's pages)."""
    import torch
    B, L, hkv, d = 64, 8192, 8, 128
    gen = torch.Generator(device="cuda").manual_seed(k)
    kv = [torch.randn((L // 16, hkv, 16, d), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    q = torch.randn((B * (k + 1), hq, d), generator=gen, device="cuda").bfloat16()
    table = torch.arange(L // 16, dtype=torch.int32, device="cuda").repeat(B, 1)
    spec = torch.full((B,), k, dtype=torch.int32, device="cuda")
    outs = []
    for others in (L, 300):
        ctx = torch.full((B,), others, dtype=torch.int32, device="cuda")
        ctx[B // 2] = L
        out = pkg.verify_attn(q, *kv, table, ctx, spec, max_spec_len=k, out_dtype=0)
        torch.cuda.synchronize()
        outs.append(out[B // 2 * (k + 1):(B // 2 + 1) * (k + 1)].clone())
    assert torch.equal(*outs)
