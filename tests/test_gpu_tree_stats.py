"""Tree acceptance over vocabularies around the 8192-element steps of the node statistics (csrc/tree_fast.hip), with few
nodes (one step per workgroup) and many (several steps per workgroup, more requests than one scan covers), sampled, greedy
and mostly masked rows, against the CPU oracle (same bar as the other tree tests)."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_tree import _check_tree_accept, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _tree(spec, V, dtype, T, width=3, **kw):
    spec = np.asarray(spec, np.int32)
    st = W.make_custom_step(17 + V, ctx_lens=spec + 1, spec_lens=spec, vocab=V, logits_dtype=dtype, temperature=T, attention=False,
                            logits_sigma=3.0, noise_sigma=1.0, draft_temp=1.1, name=f"tree-stats-{V}", **kw)
    return W.attach_tree(st, max_width=width)


@pytest.mark.parametrize("V,dtype", [(8, "bf16"), (8184, "f16"), (8192, "bf16"), (8200, "bf16"), (16392, "f16"), (128256, "bf16"),
                                     (262152, "bf16"), (524288, "f16")])
def test_tree_accept_around_the_steps(V, dtype, oracle_mod, pkg):  # noqa: F811
    _check_tree_accept(_tree([3, 0, 5, 1], V, dtype, [0.8, 1.0, 1.0, 0.0]), oracle_mod, pkg)


@pytest.mark.parametrize("B,V", [(420, 24592), (1300, 8200)])
def test_tree_accept_many_nodes(B, V, oracle_mod, pkg):  # noqa: F811
    rng = np.random.default_rng(B)
    T = rng.choice(np.array([0.0, 0.7, 1.0], np.float32), B)
    _check_tree_accept(_tree(rng.integers(0, 5, B), V, "bf16", T), oracle_mod, pkg)


def test_tree_accept_masked_rows(oracle_mod, pkg):  # noqa: F811
    _check_tree_accept(_tree([4, 2, 6], 16392, "bf16", [0.9, 1.0, 0.0], masked_frac=0.95), oracle_mod, pkg)


@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("T,offset", [(0.8, 60.0), (0.8, -60.0), (1.0, -40.0), (1.0, 0.0)])
def test_tree_accept_turns_where_the_ratio_is(dtype, T, offset, pkg):  # noqa: F811
    """One child per root, uniforms a hair below and above p / q: logits far from zero must not move p.

    Bound: the argument of the exponential, (l - m) / T * log2(e) of magnitude at most 8, is rounded twice (2.4e-7 each, times
    ln 2); exponential, reciprocal of the normaliser, product and quotient 1.2e-7 at most each, of which two are half that;
    fp32 sums of 32 terms in the normaliser 1e-7; the uniform 6e-8: 1e-6 in all. Tested 1.3e-6 away from the ratio."""
    import torch
    B, V = 256, 8192
    dt = getattr(torch, dtype)
    gen = torch.Generator(device="cuda").manual_seed(7)
    logits = (3.0 * torch.randn((2 * B, V), generator=gen, device="cuda") + offset).to(dt)
    p = torch.softmax(logits[0::2].double() / T, dim=1)
    i = torch.arange(B, device="cuda")
    x = p.topk(8, dim=1).indices[i, i % 8]
    q = torch.zeros((B, V), dtype=dt, device="cuda")
    q[i, x] = (p[i, x] / 0.7).to(dt)
    ratio = p[i, x] / q[i, x].double()
    parents = torch.tensor([-1, 0] * B, dtype=torch.int32, device="cuda")
    spec, temp = torch.ones(B, dtype=torch.int32, device="cuda"), torch.full((B,), T, device="cuda")
    for side in (-1.3e-6, 1.3e-6):
        uni = torch.zeros((2 * B, 2), device="cuda")
        uni[0::2, 0] = (ratio * (1.0 + side)).float()
        accepted = pkg.accept_tree(logits, q, x.int(), parents, uni, spec, temp, max_spec_len=1)[1]
        torch.cuda.synchronize()
        assert int((accepted == 1).sum()) == (B if side < 0 else 0), side


def test_tree_accept_at_temperatures_next_to_zero(oracle_mod, pkg):  # noqa: F811
    _check_tree_accept(_tree([3, 5, 2, 6, 1], 8200, "bf16", [1e-8, 1e-10, 1e-7, 1e-9, 1e-6]), oracle_mod, pkg)
