"""The binding's native call path (csrc_python/fastcall.cpp) against the Python one it stands in for: same results, same
errors, same treatment of everything that is not a plain call."""
import types

import pytest

import paper_2503_05096_amd as pkg
import workloads as W
from paper_2503_05096_amd import binding
from workloads.device import to_device

NAMES = ("verify_attn", "accept", "accept_tree", "kv_append", "kv_compact_path", "commit", "draft_sample")


@pytest.fixture
def python_only(monkeypatch):
    """call(f): f() with the native path switched off"""
    off = types.SimpleNamespace(**{n: lambda *a: NotImplemented for n in NAMES})

    def call(f):
        with monkeypatch.context() as m:
            m.setattr(binding, "_fast", off)
            return f()
    return call


def test_what_is_not_plain_is_left_to_python():
    import torch
    fast = binding._native()
    t = torch.zeros(2, 2)                                                  # not on a GPU
    assert fast.kv_append(t, t, t, t, t, t, t, 3, None) is NotImplemented
    assert fast.verify_attn(*[t] * 6, None, 3, 0.0, None, "run", None, None, None) is NotImplemented
    assert fast.accept(*[t] * 6, 3, None, None, None, None, None) is NotImplemented
    for n in NAMES:
        assert getattr(fast, n)() is NotImplemented                        # wrong number of arguments
    with pytest.raises(AssertionError):
        pkg.kv_append(t.view(2, 2, 1), t.view(2, 2, 1), t.view(1, 2, 2, 1), t.view(1, 2, 2, 1), t.int(), t.int(), t.int(),
                      max_spec_len=3)


def _flat(r):
    return [] if r is None else [x for x in (r if isinstance(r, tuple) else (r,)) if x is not None]


@pytest.mark.gpu
def test_native_calls_equal_python_calls(python_only):
    import torch
    st = W.attach_tree(W.make_custom_step(11, ctx_lens=[70, 300, 33], spec_lens=[2, 0, 4], n_q_heads=8, n_kv_heads=2, head_dim=128,
                                          dtype="bf16", vocab=2048, logits_dtype="bf16", temperature=[0.8, 1.0, 0.0]), max_width=2)
    d = to_device(st)
    k = st.max_spec_len
    at = (d.q, d.k_pages, d.v_pages, d.block_table, d.ctx_lens, d.spec_lens)
    rows = (d.target_logits, d.draft_probs, d.draft_tokens)
    tail = (d.uniforms, d.spec_lens, d.temperature)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    new = torch.randn(st.total_q, 2, 128, device="cuda").bfloat16()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    toks, lens, path = pkg.accept_tree(*rows, d.parents, *tail, max_spec_len=k)

    def appended(f):
        kp, vp = d.k_pages.clone(), d.v_pages.clone()
        f(kp, vp)
        return kp, vp
    calls = {
        "attn": lambda: pkg.verify_attn(*at, max_spec_len=k),
        "attn f32 out": lambda: pkg.verify_attn(*at, max_spec_len=k, out_dtype=0, scale=0.1),
        "attn out given": lambda: pkg.verify_attn(*at, torch.empty_like(d.q), max_spec_len=k, workspace=ws),
        "attn tree": lambda: pkg.verify_attn(*at, max_spec_len=k, parents=d.parents),
        "attn plan": lambda: (pkg.verify_attn(*at, max_spec_len=k, plan="build", workspace=ws),
                              pkg.verify_attn(*at, max_spec_len=k, plan="reuse", workspace=ws)),
        "attn stream": lambda: pkg.verify_attn(*at, max_spec_len=k, workspace=ws, stream=side),
        "attn vector": lambda: pkg.verify_attn(*at, max_spec_len=k, path="vector"),
        "accept": lambda: pkg.accept(*rows, *tail, max_spec_len=k),
        "accept wide": lambda: pkg.accept(*rows, *tail, max_spec_len=k, out_stride=k + 4),
        "accept no drafts": lambda: pkg.accept(d.target_logits[:3], None, None, d.uniforms[:3], torch.zeros_like(d.spec_lens),
                                               d.temperature, max_spec_len=0),
        "tree": lambda: pkg.accept_tree(*rows, d.parents, *tail, max_spec_len=k),
        "append": lambda: appended(lambda kp, vp: pkg.kv_append(new, new, kp, vp, *at[3:], max_spec_len=k)),
        "compact": lambda: appended(lambda kp, vp: pkg.kv_compact_path(kp, vp, *at[3:], path, lens, max_spec_len=k)),
        "commit": lambda: pkg.commit(toks, lens, d.spec_lens, d.ctx_lens, max_spec_len=k),
        "commit next": lambda: pkg.commit(toks, lens, d.spec_lens, d.ctx_lens, max_spec_len=k, next_spec_lens=d.spec_lens),
        "commit seq": lambda: (lambda seq, n: (*pkg.commit(toks, lens, d.spec_lens, d.ctx_lens, max_spec_len=k, seq_tokens=seq,
                                                           seq_lens=n), seq, n))(torch.zeros(3, 9, dtype=torch.int32, device="cuda"),
                                                                                 torch.ones(3, dtype=torch.int32, device="cuda")),
        "draft": lambda: pkg.draft_sample(d.target_logits[:3], d.temperature, d.uniforms[:3, 0].contiguous()),
        "draft f32": lambda: pkg.draft_sample(d.target_logits[:3].float(), d.temperature, d.uniforms[:3, 0].contiguous(),
                                              probs_dtype=torch.float16),
        "draft rows": lambda: pkg.draft_sample(d.target_logits[:3], d.temperature, d.uniforms[:3, 0].contiguous(),
                                               draft_probs=torch.zeros(5, 2048, device="cuda"),
                                               out_rows=torch.tensor([4, 0, 2], dtype=torch.int32, device="cuda")),
    }
    for name, f in calls.items():
        a = _flat(f())
        torch.cuda.synchronize()
        b = _flat(python_only(f))
        torch.cuda.synchronize()
        assert len(a) == len(b), name
        for x, y in zip(a, b):
            assert x.dtype == y.dtype and x.shape == y.shape and x.device == y.device, name
            assert torch.equal(x.view(torch.uint8) if x.dtype.is_floating_point else x,
                               y.view(torch.uint8) if y.dtype.is_floating_point else y), name


@pytest.mark.gpu
def test_native_calls_raise_what_python_calls_raise(python_only):
    import torch
    st = W.make_custom_step(12, ctx_lens=[40], spec_lens=[1], n_q_heads=2, n_kv_heads=2, head_dim=64, dtype="bf16", vocab=1024,
                            logits_dtype="bf16")
    d = to_device(st)
    at = [d.q, d.k_pages, d.v_pages, d.block_table, d.ctx_lens, d.spec_lens]
    bad = {
        "dtype of the lengths": lambda: pkg.verify_attn(*at[:4], d.ctx_lens.long(), at[5], max_spec_len=1),
        "not contiguous": lambda: pkg.verify_attn(d.q.transpose(0, 1), *at[1:], max_spec_len=1),
        "two types": lambda: pkg.verify_attn(d.q.half(), *at[1:], max_spec_len=1),
        "unsupported head dim": lambda: pkg.verify_attn(d.q[:, :, :4].contiguous(), d.k_pages[..., :4].contiguous(),
                                                        d.v_pages[..., :4].contiguous(), *at[3:], max_spec_len=1),
        "rows beyond the bound": lambda: pkg.verify_attn(*at, max_spec_len=0),
        "plan without workspace": lambda: pkg.verify_attn(*at, max_spec_len=1, plan="reuse"),
        "small workspace": lambda: pkg.verify_attn(*at, max_spec_len=1, workspace=torch.empty(256, dtype=torch.uint8, device="cuda")),
        "unknown path": lambda: pkg.verify_attn(*at, max_spec_len=1, path="quick"),
        "uniforms in fp64": lambda: pkg.accept(d.target_logits, d.draft_probs, d.draft_tokens, d.uniforms.double(), d.spec_lens,
                                               d.temperature, max_spec_len=1),
        "narrow outputs": lambda: pkg.accept(d.target_logits, d.draft_probs, d.draft_tokens, d.uniforms, d.spec_lens, d.temperature,
                                             max_spec_len=1, out_stride=1),
        "odd vocabulary": lambda: pkg.draft_sample(d.target_logits[:, :1001].contiguous(), torch.ones(2, device="cuda"),
                                                   torch.zeros(2, device="cuda")),
    }
    for name, f in bad.items():
        with pytest.raises(Exception) as a:
            f()
        with pytest.raises(type(a.value)) as b:
            python_only(f)
        assert str(a.value) == str(b.value), name
