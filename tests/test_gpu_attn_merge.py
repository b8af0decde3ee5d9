"""Direct attention calls whose splits are merged in the main kernel by whoever finishes last: at the edges of the splits,
against the oracle; in any workspace whatever it holds; in a captured graph, whose launches find what the replay before
left."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.harness import to_device
from tests.test_gpu_parity import check_attention, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

MERGED = [         # ctx_lens, spec_lens, Hq, Hkv, d, dtype, possible splits; the longest context fills the last one, or nearly
          ([512, 511, 257, 256, 1], [3, 0, 2, 1, 0], 8, 2, 128, "bf16", 2), ([700, 600, 31], [1, 3, 0], 8, 2, 128, "f16", 3),
          ([1024, 769], [3, 2], 8, 2, 128, "f16", 4),
          ([900, 31, 513, 6], [7, 7, 2, 0], 32, 8, 64, "bf16", 2), ([1500, 1000], [5, 3], 64, 16, 64, "f16", 3), ([2048, 1025], [3, 0], 64, 16, 64, "bf16", 4),
          ([512, 128, 129, 400], [4, 1, 2, 0], 8, 8, 64, "f32", 4), ([250, 380], [7, 6], 8, 2, 64, "f32", 3),
          ([512, 100], [3, 1], 8, 2, 128, "f32", 4), ([256, 129, 7], [0, 2, 3], 8, 2, 128, "f32", 2)]
APART = [          # one split too many, or two row tiles of 128 channels: the combine kernel
         ([1040], [3], 8, 2, 128, "bf16", 5), ([2064, 40], [1, 2], 8, 2, 64, "f16", 5), ([520], [4], 8, 8, 64, "f32", 5),
         ([600, 513], [7, 5], 8, 2, 128, "bf16", 3), ([380], [7], 8, 2, 128, "f32", 3)]


def name(s):
    return f"B{len(s[0])}-L{max(s[0])}-{s[2]}x{s[3]}-{s[5]}-{s[4]}-{s[6]}"


def step(shape):
    ctx, spec, hq, hkv, d, dtype, _ = shape
    return W.make_custom_step(len(ctx) + d, ctx_lens=ctx, spec_lens=spec, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                              acceptance=False, name=f"merge-{dtype}-{d}")


def own_workspace(shape, dev, pkg):  # noqa: F811
    """A workspace, its flag words (a word per unit and wavefront, at its end), an output and the call."""
    args = [dev.q, dev.k_pages, dev.v_pages, dev.block_table, dev.ctx_lens, dev.spec_lens]
    k = max(shape[1])
    dims = pkg.attn_dims(args[0], args[1], args[3], max_spec_len=k)
    ws = torch.empty(pkg.lib().adaspec_verify_attn_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    nbytes = -(-len(shape[0]) * shape[6] * shape[3] * 32 // 256) * 256
    out = torch.empty_like(dev.q)
    return ws, ws[-nbytes:], out, args, lambda: pkg.verify_attn(*args, max_spec_len=k, workspace=ws, out=out)


@pytest.mark.parametrize("shape", MERGED + APART, ids=name)
def test_splits_merged_in_the_kernel(shape, oracle_mod, pkg):  # noqa: F811
    check_attention(step(shape), oracle_mod, pkg)


@pytest.mark.parametrize("shape", MERGED, ids=name)
def test_leftovers_in_the_workspace(shape, pkg):  # noqa: F811
    dev = to_device(step(shape), acceptance=False)
    ws, flags, out, args, call = own_workspace(shape, dev, pkg)
    want = pkg.verify_attn(*args, max_spec_len=max(shape[1]))
    for fill in (0, 255, None, 127, None, None):
        out.zero_()
        if fill is not None:
            ws.fill_(fill)
        call()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        if fill == 0:
            assert not flags.any()              # every mark has been taken back


@pytest.mark.parametrize("shape", MERGED, ids=name)
def test_replays_in_a_row(shape, pkg):  # noqa: F811
    """A captured launch puts the same mark down every time, and nothing but replays touches its workspace: the mark of the
    replay before must be gone. Other inputs and other lengths, so other numbers of splits, every time."""
    dev = to_device(step(shape), acceptance=False)
    ws, flags, out, args, call = own_workspace(shape, dev, pkg)
    k = max(shape[1])
    ws.zero_()
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    rng = np.random.default_rng(len(shape[0]) + shape[4])
    most, least = np.array(shape[0]), np.minimum(np.array(shape[0]), np.array(shape[1]) + 1)
    gen = torch.Generator(device="cuda").manual_seed(shape[4])
    for i in range(12):
        ctx = (most, least, most, rng.integers(least, most + 1))[i % 4]
        dev.ctx_lens.copy_(torch.tensor(ctx, dtype=torch.int32))
        for t in (dev.q, dev.k_pages, dev.v_pages):
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, pkg.verify_attn(*args, max_spec_len=k)), (i, ctx)      # (in the library's own workspace)
        assert not flags.any(), (i, ctx)
