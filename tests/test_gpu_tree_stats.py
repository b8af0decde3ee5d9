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
