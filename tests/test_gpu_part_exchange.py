"""Workgroups that share a row take each other's sums where they come in time and compute them otherwise
(csrc/part_exchange.h): a library whose workgroups never wait gives the same results bit for bit."""
import os

import numpy as np
import pytest

import workloads as W
from workloads.device import to_device
from paper_2503_05096_amd import binding, build
from tests.test_gpu_tree import _check_tree_accept, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
IMPATIENT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libadaspec_impatient.so")


@pytest.fixture
def impatient(monkeypatch):
    """Calls go to the library that never waits (through ctypes) until the returned function switches back."""
    if not os.path.exists(IMPATIENT):
        build.build_library()
        build.build_impatient(IMPATIENT)
    L = binding._open(IMPATIENT)

    def run(call):
        with monkeypatch.context() as m:
            m.setattr(binding, "_lib", L)
            m.setattr(binding, "_fast", binding._PythonOnly())
            return call()
    return run


def _tree(spec, V, dtype, T, **kw):
    spec = np.asarray(spec, np.int32)
    st = W.make_custom_step(31 + V, ctx_lens=spec + 1, spec_lens=spec, vocab=V, logits_dtype=dtype, temperature=T, attention=False,
                            logits_sigma=3.0, noise_sigma=1.5, draft_temp=1.3, name=f"tree-exchange-{V}", **kw)
    return W.attach_tree(st, max_width=4)


# parts of one step and of four, a last part that is nearly empty, one of a single step; draws in every part; 16 and 8 parts
@pytest.mark.parametrize("B,V,dtype", [(4, 128256, "bf16"), (40, 128256, "f16"), (40, 98312, "bf16"), (70, 131072, "bf16"),
                                       (5, 262152, "f16"), (30, 262144, "bf16"), (3, 524288, "bf16"), (60, 40968, "bf16")])
def test_tree_walk_without_waiting(B, V, dtype, oracle_mod, pkg, impatient):  # noqa: F811
    import torch
    rng = np.random.default_rng(V + B)
    T = rng.choice(np.array([0.0, 0.7, 1.0, 1.0], np.float32), B)
    st = _tree(rng.integers(0, 7, B), V, dtype, T)
    _, want = _check_tree_accept(st, oracle_mod, pkg)
    dev = to_device(st, attention=False)

    def call():
        got = pkg.accept_tree(dev.target_logits, dev.draft_probs, dev.draft_tokens, dev.parents, dev.uniforms, dev.spec_lens,
                              dev.temperature, max_spec_len=st.max_spec_len)
        torch.cuda.synchronize()
        return got
    assert all(torch.equal(a, b) for a, b in zip(want, impatient(call)))
