"""Workgroups that share a row take each other's sums where they come in time and compute them otherwise
(csrc/part_exchange.h): libraries whose workgroups never wait, or not for some words, give the same results bit for bit."""
import numpy as np
import pytest

import workloads as W
from workloads.device import to_device
from paper_2503_05096_amd import binding
from tests import exchange_builds
from tests.test_gpu_parity import check_accept
from tests.test_gpu_tree import _check_tree_accept, pkg  # noqa: F401  (fixture)
from workloads.verify_step import _store, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(params=sorted(exchange_builds.DEFINES))
def impatient(request, monkeypatch):
    """Calls go to a library that never waits, or not for some words (through ctypes), until the returned function switches back."""
    L = binding._open(exchange_builds.ensure(request.param))

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


def _draft_inputs(R, V, dtype, seed, T=None, lead_masked=False):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = 3.0 * torch.randn((R, V), generator=gen, device="cuda")
    if lead_masked:                                 # threads and parts without a finite logit, logits far apart
        x[::2, :V // 2] = -float("inf")
        x[1::2] = torch.where(torch.rand((R // 2, V), generator=gen, device="cuda") < 0.5, x[1::2] - 300.0, x[1::2] + 300.0)
    t = torch.tensor([0.8, 0.0, 1.0, 1e-8], device="cuda").repeat(R)[:R] if T is None else torch.full((R,), T, device="cuda")
    return x.to(dtype), t, torch.rand(R, generator=gen, device="cuda")


# whole rows, parts of every length, a last part that is nearly empty, 1024 threads, the most parts; all pairs of element sizes
@pytest.mark.parametrize("R,V,ldt,pdt", [(4, 16384, "bfloat16", "bfloat16"), (6, 32776, "bfloat16", "float32"), (5, 128256, "float16", "float16"),
                                         (128, 128256, "bfloat16", "bfloat16"), (70, 65544, "bfloat16", "float16"), (4, 524288, "float32", "float32"),
                                         (40, 50184, "float32", "bfloat16"), (2, 262152, "float16", "bfloat16"), (160, 65536, "bfloat16", "bfloat16")])
@pytest.mark.parametrize("lead_masked", [False, True])
def test_draft_rows_without_waiting(R, V, ldt, pdt, lead_masked, pkg, impatient):  # noqa: F811
    import torch
    x, t, u = _draft_inputs(R, V, getattr(torch, ldt), R + V, lead_masked=lead_masked)

    def call():
        got = pkg.draft_sample(x, t, u, probs_dtype=getattr(torch, pdt))
        torch.cuda.synchronize()
        return got
    want = call()
    assert all(torch.equal(a, b) for a, b in zip(want, impatient(call)))
    q = torch.softmax(x.double() / torch.where(t > 0, t.double(), 1.0)[:, None], dim=1)
    ulp = {"float32": 2e-5, "float16": 2.0 ** -10, "bfloat16": 2.0 ** -7}[pdt]      # (a step of the stored type, fp32: bar of the draft tests)
    assert bool(((want[0].double() - q).abs() <= ulp * q + 1e-7).all())
    assert torch.equal(want[2], want[0].float().gather(1, want[1].long()[:, None])[:, 0])
    assert torch.equal(want[1][t == 0].long(), x[t == 0].float().argmax(1))


def _bits(t):
    import torch
    return t.view({2: torch.int16, 4: torch.int32}[t.element_size()])


@pytest.mark.parametrize("V,dtype", [(32776, "bfloat16"), (128256, "float16"), (262152, "bfloat16"), (50184, "float32")])
def test_draft_rows_with_a_nan_without_waiting(V, dtype, pkg, impatient):  # noqa: F811
    import torch
    x, t, u = _draft_inputs(8, V, getattr(torch, dtype), V)
    x[4:, 4096:V - 4096] = -float("inf")             # (NaNs beside finite logits of their thread, and beside masked ones only)
    for r, i in enumerate([3, V // 2, V - 1, V // 3] * 2):
        _bits(x)[r, i] = -1 if r % 2 else 0x7fff * (65537 if dtype == "float32" else 1)

    def call():
        got = pkg.draft_sample(x, t, u)
        torch.cuda.synchronize()
        return got
    want, got = call(), impatient(call)
    assert bool(torch.isnan(want[0].float()).all()) and bool(torch.isnan(got[0].float()).all())
    assert torch.equal(want[1], got[1]) and torch.equal(want[2].nan_to_num(-1.0), got[2].nan_to_num(-1.0))


@pytest.mark.parametrize("V,dtype", [(32776, "bfloat16"), (128256, "bfloat16"), (262152, "float16")])
def test_draft_rows_masked_with_the_lowest_number_without_waiting(V, dtype, pkg, impatient):  # noqa: F811
    import torch
    x, t, u = _draft_inputs(8, V, getattr(torch, dtype), V + 1)
    x[:, V // 4:V // 2] = torch.finfo(x.dtype).min
    x[:, V - 512:] = torch.finfo(x.dtype).min

    def call():
        got = pkg.draft_sample(x, t, u)
        torch.cuda.synchronize()
        return got
    want = call()
    assert bool(torch.isfinite(want[0].float()).all()) and bool((want[2][t > 0] > 0).all())
    assert all(torch.equal(a, b) for a, b in zip(want, impatient(call)))


@pytest.mark.parametrize("V,ldt", [(8200, "bf16"), (12288, "bf16"), (128256, "f32")])
def test_accept_rows_masked_with_the_lowest_number_without_waiting(V, ldt, oracle_mod, pkg, impatient):  # noqa: F811
    import torch
    st = _accept_step(20, V, ldt, ldt, 700 + V)
    lowest = np.uint16(0xFF7F) if ldt == "bf16" else np.finfo(np.float32).min
    st.target_logits[:, V // 4:3 * V // 4] = lowest
    st.target_logits[:, V - 512:] = lowest
    check_accept(st, oracle_mod, pkg)
    dev = to_device(st, attention=False)

    def call():
        got = pkg.accept(dev.target_logits, dev.draft_probs, dev.draft_tokens, dev.uniforms, dev.spec_lens, dev.temperature,
                         max_spec_len=st.max_spec_len)
        torch.cuda.synchronize()
        return got
    assert all(torch.equal(a, b) for a, b in zip(call(), impatient(call)))


@pytest.mark.parametrize("R,V,dtype", [(5, 128256, "bfloat16"), (3, 262144, "float32")])
def test_draft_rows_in_place_without_waiting(R, V, dtype, pkg, impatient):  # noqa: F811
    """Rows over their own logits (and, in the same call, one beside them): nobody reads what another workgroup has overwritten."""
    import torch
    x, t, u = _draft_inputs(R, V, getattr(torch, dtype), R)
    want = [v.clone() for v in pkg.draft_sample(x, t, u)]
    buffer = torch.zeros((R + 2, V), dtype=x.dtype, device="cuda")
    rows = torch.arange(1, R + 1, dtype=torch.int32, device="cuda")
    rows[R - 1] = R + 1                                          # (the last row's logits are at row R)

    def call():
        buffer[1:R + 1] = x
        got = pkg.draft_sample(buffer[1:R + 1], t, u, draft_probs=buffer, out_rows=rows)
        torch.cuda.synchronize()
        return got[0][rows.long()].clone(), got[1], got[2]
    for got in (call(), impatient(call)):
        assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("V,ldt", [(8200, "bf16"), (12288, "f16"), (50272, "f32")])
def test_accept_bonus_rows_with_a_nan_without_waiting(V, ldt, pkg, impatient):  # noqa: F811
    """A NaN beside the only finite logits of its part: whoever computes the part must find the same maximum."""
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[ldt]
    gen = torch.Generator(device="cuda").manual_seed(V)
    x = (3.0 * torch.randn((6, V), generator=gen, device="cuda")).to(dt)
    x[:, V // 2:] = -float("inf")
    x[:, V - 16:V - 8] = 1.0
    _bits(x)[:, V - 12] = 0x7fff * (65537 if ldt == "f32" else 1)
    T = torch.tensor([0.7, 1.0, 0.0, 1.0, 1.3, 0.7], device="cuda")
    zeros = torch.zeros(6, dtype=torch.int32, device="cuda")

    def call():
        got = pkg.accept(x, torch.zeros((0, V), dtype=dt, device="cuda"), zeros[:0], torch.full((6, 2), 0.999, device="cuda"), zeros, T,
                         max_spec_len=2, path="auto" if ldt == "f32" else "two_pass")
        torch.cuda.synchronize()
        return got
    assert all(torch.equal(a, b) for a, b in zip(call(), impatient(call)))


@pytest.mark.parametrize("R,V", [(3, 50272), (128, 128256)])
def test_draft_rows_replayed_from_a_hip_graph(R, V, pkg):  # noqa: F811
    """A captured launch keeps its mark: every replay, on other inputs, must not find what the one before has left."""
    import torch
    sets = [_draft_inputs(R, V, torch.bfloat16, s, 0.8) for s in range(4)]
    x, t, u = (v.clone() for v in sets[0])
    want = [[v.clone() for v in pkg.draft_sample(*s)] for s in sets]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = pkg.draft_sample(x, t, u)
    for turn in range(2):
        for s, w in zip(sets, want):
            for dst, src in zip((x, t, u), s):
                dst.copy_(src)
            graph.replay()
            if turn:                                # an eager call in between, with a mark of its own
                pkg.draft_sample(*sets[0])
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, w))


def _replay(call, inputs, sets, want, between):
    """Captures call() on `inputs` and replays it on every set, with eager calls in between."""
    import torch
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = call()
    for turn in range(2):
        for s, w in zip(sets, want):
            for dst, src in zip(inputs, s):
                dst.copy_(src)
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, w))
            if turn:
                between()


@pytest.mark.parametrize("R,V", [(3, 50272), (128, 128256), (20, 262144)])
def test_draft_rows_replayed_without_waiting(R, V, pkg, impatient):  # noqa: F811
    """Like the replays above, by workgroups that give up on words, with eager calls of other rows and vocabularies (words laid out
    otherwise) on the same workspace in between."""
    import torch
    sets = [_draft_inputs(R, V, torch.bfloat16, s, 0.8) for s in range(3)]
    x, t, u = (v.clone() for v in sets[0])
    want = [[v.clone() for v in pkg.draft_sample(*s)] for s in sets]
    others = [_draft_inputs(r, v, torch.bfloat16, 9, 1.0) for r, v in ((5, 128256), (70, 65544), (2, 524288))]
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    eager = iter(others * 2)

    def between():
        o = next(eager)
        pkg.draft_sample(*o, workspace=ws)                       # (its words carry the other library's marks)
        impatient(lambda: pkg.draft_sample(*o, workspace=ws))
    torch.cuda.synchronize()
    _replay(lambda: impatient(lambda: pkg.draft_sample(x, t, u, workspace=ws)), (x, t, u), sets, want, between)


@pytest.mark.parametrize("B,V,dtype", [(24, 128256, "f32"), (6, 8200, "bf16")])
def test_accept_replayed_without_waiting(B, V, dtype, pkg, impatient):  # noqa: F811
    import torch
    k = 3
    T = np.random.default_rng(B).choice(np.array([0.0, 0.7, 1.0, 1.0], np.float32), B)
    devs = [to_device(W.make_custom_step(40 + s, ctx_lens=[k + 1] * B, spec_lens=[k] * B, vocab=V, logits_dtype=dtype, temperature=T,
                                         attention=False, logits_sigma=3.0, noise_sigma=1.5, draft_temp=1.2), attention=False) for s in range(2)]
    sets = [(d.target_logits, d.draft_probs, d.draft_tokens, d.uniforms, d.spec_lens, d.temperature) for d in devs]
    call = lambda a: pkg.accept(*a, max_spec_len=k)
    want = [[v.clone() for v in call(s)] for s in sets]
    inputs = tuple(v.clone() for v in sets[0])
    torch.cuda.synchronize()
    _replay(lambda: impatient(lambda: call(inputs)), inputs, sets, want, lambda: None)


def test_tree_walk_replayed_without_waiting(pkg, impatient):  # noqa: F811
    import torch
    B, V, k = 12, 128256, 4
    steps = [_tree([k] * B, V, "bf16", np.full(B, 0.9, np.float32)) for _ in range(2)]
    devs = [to_device(st, attention=False) for st in steps]
    sets = [(d.target_logits, d.draft_probs, d.draft_tokens, d.parents, d.uniforms, d.spec_lens, d.temperature) for d in devs]
    sets[1] = tuple(v.clone() for v in sets[1])
    sets[1][4].copy_(1.0 - sets[1][4])                           # other decisions and other draws
    call = lambda a: pkg.accept_tree(*a, max_spec_len=k)
    want = [[v.clone() for v in call(s)] for s in sets]
    inputs = tuple(v.clone() for v in sets[0])
    torch.cuda.synchronize()
    _replay(lambda: impatient(lambda: call(inputs)), inputs, sets, want, lambda: None)


def _accept_step(B, V, ldt, pdt, seed, equal=False, **kw):
    rng = np.random.default_rng(seed)
    spec = rng.integers(0, 6, B).astype(np.int32)
    T = rng.choice(np.array([0.0, 0.7, 1.0, 1.0], np.float32), B)
    st = W.make_custom_step(seed, ctx_lens=spec + 1, spec_lens=spec, vocab=V, logits_dtype=ldt, temperature=T, attention=False,
                            logits_sigma=3.0, noise_sigma=1.5, draft_temp=1.2, name=f"accept-exchange-{B}-{V}", **kw)
    if equal:                                       # p == q and tokens that are rejected all the same: no residual mass, drawn from p
        st.target_logits = np.zeros_like(st.target_logits)
        st.draft_probs = _store(np.full(st.draft_probs.shape, 1.5 / V, np.float32), ldt)
    if pdt != ldt:
        st.draft_probs = _store(to_f64(st.draft_probs, ldt).astype(np.float32), pdt)
        st.probs_dtype = pdt
    return st


# one part, parts of every length, a last part that is nearly empty, the most parts, more parts than fit the chip at once; rows that have gone back to many small workgroups (32008, 50272)
@pytest.mark.parametrize("B,V,ldt,pdt", [(5, 2000, "f32", "f32"), (64, 128256, "f32", "f32"), (150, 32008, "f32", "bf16"), (3, 524288, "f32", "f16"),
                                         (40, 98312, "f32", "f32"), (1, 128256, "f32", "bf16"), (200, 50272, "f32", "f32"), (100, 114704, "f32", "f32"),
                                         (6, 12288, "bf16", "bf16"), (70, 8200, "f16", "f32"), (300, 4104, "bf16", "f16")])
@pytest.mark.parametrize("kind", ["", "masked", "equal"])
def test_accept_without_waiting(B, V, ldt, pdt, kind, oracle_mod, pkg, impatient):  # noqa: F811
    import torch
    st = _accept_step(B, V, ldt, pdt, 500 + B, equal=kind == "equal", **({"masked_frac": 0.99} if kind == "masked" else {}))
    if kind != "equal" or V == 32008:
        check_accept(st, oracle_mod, pkg)
    dev = to_device(st, attention=False)

    def call():
        got = pkg.accept(dev.target_logits, dev.draft_probs, dev.draft_tokens, dev.uniforms, dev.spec_lens, dev.temperature,
                         max_spec_len=st.max_spec_len)
        torch.cuda.synchronize()
        return got
    assert all(torch.equal(a, b) for a, b in zip(call(), impatient(call)))
