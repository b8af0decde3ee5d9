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


@pytest.mark.parametrize("ldt,pdt", [("bf16", "f32"), ("f16", "bf16"), ("bf16", "bf16"), ("f16", "f16"), ("f32", "f32"), ("f32", "bf16")])
@pytest.mark.parametrize("T,offset,V", [(0.8, 60.0, 32000), (0.8, -60.0, 32000), (1.0, -40.0, 8192), (1.0, 0.0, 128256)])
def test_accept_parts_turn_where_the_ratio_is(ldt, pdt, T, offset, V, pkg):  # noqa: F811
    """One draft per request, uniforms a hair below and above p / q: logits far from zero must not move p.

    Bound: exponential, reciprocal of the normaliser, product and quotient 1.2e-7 at most each, of which two are half that;
    fp32 sums of up to 512 terms per thread in the normaliser 3e-7; log2(e) / T rounded in fp32 1.2e-7 of the exponent, which
    is 5 away from its mean at most: 4e-7; the uniform 6e-8: 1.2e-6 in all. Tested 1.3e-6 away from the ratio."""
    import torch
    dts = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
    B, dt = 192, dts[ldt]
    gen = torch.Generator(device="cuda").manual_seed(7)
    logits = (3.0 * torch.randn((2 * B, V), generator=gen, device="cuda") + offset).to(dt)
    p = torch.softmax(logits[0::2].double() / T, dim=1)
    i = torch.arange(B, device="cuda")
    x = p.topk(8, dim=1).indices[i, i % 8]
    q = torch.zeros((B, V), dtype=dts[pdt], device="cuda")
    q[i, x] = (p[i, x] / 0.7).to(q.dtype)
    ratio = p[i, x] / q[i, x].double()
    spec, temp = torch.ones(B, dtype=torch.int32, device="cuda"), torch.full((B,), T, device="cuda")
    for side in (-1.3e-6, 1.3e-6):
        uni = torch.zeros((2 * B, 2), device="cuda")
        uni[0::2, 0] = (ratio * (1.0 + side)).float()
        accepted = pkg.accept(logits, q, x.int(), uni, spec, temp, max_spec_len=1)[1]
        torch.cuda.synchronize()
        assert int((accepted == 1).sum()) == (B if side < 0 else 0), side


@pytest.mark.parametrize("ldt,pdt", [("bf16", "f32"), ("f16", "f32"), ("f16", "bf16"), ("f32", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("offset", [0.0, 40.0])
def test_accept_parts_at_temperatures_next_to_zero(ldt, pdt, offset, oracle_mod, pkg):  # noqa: F811
    """Temperatures that stand for 'greedy' without being 0: scaled logits up to 1e12."""
    st = _step(4096, ldt, pdt, spec=[3, 0, 2, 6, 1, 4], temp=[1e-8, 1e-10, 1e-7, 1e-9, 1e-6, 1e-10])
    st.target_logits = _store((to_f64(st.target_logits, ldt) + offset).astype(np.float32), ldt)
    check_accept(st, oracle_mod, pkg)


@pytest.mark.parametrize("V", [4096, 8200, 32000, 128256])
@pytest.mark.parametrize("ldt,pdt,path", [("bf16", "bf16", "auto"), ("bf16", "bf16", "two_pass"), ("bf16", "bf16", "fast"), ("bf16", "bf16", "stream"),
                                          ("bf16", "f32", "auto"), ("f16", "f16", "auto"), ("f32", "f32", "auto")])
def test_accept_rows_masked_with_the_lowest_number(ldt, pdt, path, V, oracle_mod, pkg):  # noqa: F811
    """Masked by the type's lowest number in place of -inf, alone and in stretches (threads, parts of which nothing else is left): a
    product of it with log2(e) / T overflows for bf16."""
    st = _step(V, ldt, pdt, spec=[3, 0, 2, 6, 1, 0], temp=[0.8, 1.0, 0.0, 0.5, 0.0, 0.7], masked_frac=0.3)
    x = to_f64(st.target_logits, ldt)
    gone = np.isneginf(x)
    gone[:, V // 4:V // 2] = True
    gone[:, V - 256:] = True
    st.target_logits[gone] = {"f32": np.finfo(np.float32).min, "f16": np.finfo(np.float16).min, "bf16": np.uint16(0xFF7F)}[ldt]
    st.draft_probs[:, V // 4:V // 2] = 0
    check_accept(st, oracle_mod, pkg, path=path)
    st.temperature[:] = np.array([100.0, 30.0, 0.0, 3.0, 300.0, 50.0], np.float32)      # the product is finite, but coarse
    check_accept(st, oracle_mod, pkg, path=path)
    if ldt == "f16":
        st.temperature[:] = np.array([1e-5, 1e-6, 0.0, 1e-6, 1e-5, 1e-6], np.float32)
        check_accept(st, oracle_mod, pkg, path=path)
