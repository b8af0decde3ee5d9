"""Acceptance in row parts (csrc/accept_parts.hip) over all pairs of storage types and up to its largest vocabulary,
through AUTO, against the CPU oracle: vocabularies around a chunk, a step of 256 chunks, a wavefront's share and a part of
1024 chunks, the largest one; sampled, greedy and masked rows, bonus rows, drafts equal to the target.

Tokens and lengths are exact except for the near-ties the oracle counts (same bar as the other acceptance tests)."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import check_accept, pkg  # noqa: F401  (fixture)
from workloads.verify_step import _store, to_f64

pytestmark = pytest.mark.gpu

TYPES = [(a, b) for a in ("f32", "f16", "bf16") for b in ("f32", "f16", "bf16")]
SPEC, TEMP = [3, 0, 2, 6, 1], [0.8, 1.0, 0.0, 1.0, 0.0]


def _step(V, ldt, pdt, spec=SPEC, temp=TEMP, **kw):
    st = W.make_custom_step(99 + V, ctx_lens=[80] * len(spec), spec_lens=spec, vocab=V, logits_dtype=ldt, temperature=temp,
                            attention=False, logits_sigma=3.0, draft_temp=1.1, name=f"parts-{ldt}-{pdt}-{V}",
                            **{"noise_sigma": 1.0, **kw})
    if pdt != ldt:
        st.draft_probs = _store(to_f64(st.draft_probs, ldt).astype(np.float32), pdt)
        st.probs_dtype = pdt
    return st


@pytest.mark.parametrize("V", [8, 1016, 1032, 4096, 8200, 32000])
@pytest.mark.parametrize("ldt,pdt", TYPES)
def test_accept_parts_types(ldt, pdt, V, oracle_mod, pkg):  # noqa: F811
    check_accept(_step(V, ldt, pdt), oracle_mod, pkg)


@pytest.mark.parametrize("V,ldt,pdt", [(128256, "f32", "f32"), (131080, "bf16", "bf16"), (262144, "f16", "f16"),
                                       (524288, "f32", "bf16"), (524288, "bf16", "f32"), (524280, "f16", "f16")])
def test_accept_parts_large_vocabularies(V, ldt, pdt, oracle_mod, pkg):  # noqa: F811
    check_accept(_step(V, ldt, pdt, spec=[2, 0, 1], temp=[0.9, 1.0, 0.0]), oracle_mod, pkg)


@pytest.mark.parametrize("ldt,pdt", [("f32", "f32"), ("bf16", "f32"), ("f32", "f16")])
def test_accept_parts_masked_rows_and_equal_distributions(ldt, pdt, oracle_mod, pkg):  # noqa: F811
    check_accept(_step(5000, ldt, pdt, masked_frac=0.9), oracle_mod, pkg)            # most logits -inf
    st = _step(2048, ldt, pdt)
    st.target_logits = _store(np.full(st.target_logits.shape, -50.0, np.float32), ldt)     # p uniform, all logits negative
    st.draft_probs = _store(np.full(st.draft_probs.shape, 1.0 / 2048, np.float32), pdt)    # q == p: no residual mass
    check_accept(st, oracle_mod, pkg)


def test_accept_beyond_the_parts_layout(oracle_mod, pkg):  # noqa: F811
    """Rows whose stride is not a multiple of 8 elements, and an odd vocabulary, stay on the portable kernel."""
    for V in (1001, 4100):
        check_accept(_step(V, "f32", "f32"), oracle_mod, pkg)
