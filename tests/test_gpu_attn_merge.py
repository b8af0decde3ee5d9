"""Direct attention calls whose splits are merged in the main kernel by whoever finishes last: at the edges of the splits,
against the oracle; in any workspace whatever it holds; in a captured graph, whose launches find what the replay before
left."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.harness import compare_attention, to_device
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [         # the longest context fills the last possible split, or nearly; (2048 and 4096: one more split than are merged)
          ([512, 511, 257, 256, 1], [3, 0, 2, 1, 0], 8, 2, 128, "bf16"), ([1024, 769], [7, 5], 8, 2, 128, "f16"),
          ([2048, 1793, 40], [3, 1, 2], 8, 2, 128, "bf16"), ([900, 31, 513], [7, 7, 2], 28, 7, 64, "bf16"),
          ([4096], [3], 4, 2, 64, "f16"), ([512, 128, 129, 400], [4, 1, 2, 0], 8, 8, 64, "f32"), ([1000, 130], [5, 6], 8, 2, 128, "f32")]


def step(shape):
    ctx, spec, hq, hkv, d, dtype = shape
    return W.make_custom_step(len(ctx) + d, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                              acceptance=False, name=f"merge-{dtype}-{d}")


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"B{len(s[0])}-L{max(s[0])}-{s[2]}x{s[3]}-{s[5]}-{s[4]}")
def test_splits_merged_in_the_kernel(shape, oracle_mod, pkg):  # noqa: F811
    check_attention(step(shape), oracle_mod, pkg)


@pytest.mark.parametrize("shape", SHAPES[::2], ids=lambda s: f"B{len(s[0])}-{s[5]}-{s[4]}")
@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
def test_leftovers_in_the_workspace(shape, graph, pkg):  # noqa: F811
    dev = to_device(step(shape), acceptance=False)
    k = max(shape[1])
    args = [dev.q, dev.k_pages, dev.v_pages, dev.block_table, dev.ctx_lens, dev.spec_lens]
    want = pkg.verify_attn(*args, max_spec_len=k)
    dims = pkg.attn_dims(args[0], args[1], args[3], max_spec_len=k)
    ws = torch.empty(pkg.lib().adaspec_verify_attn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(want)
    call = lambda: pkg.verify_attn(*args, max_spec_len=k, workspace=ws, out=out)  # noqa: E731
    if graph:
        call()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call()
    for fill in (0, 255, None, 127, None, None):
        out.zero_()
        if fill is not None:
            ws.fill_(fill)
        g.replay() if graph else call()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        call()                                  # an eager call between the replays
        torch.cuda.synchronize()
        assert torch.equal(out, want)
