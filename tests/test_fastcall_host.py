"""The native call path (csrc_python/fastcall.cpp) where no GPU is needed: a build of it that takes meta tensors, with
functions of this file in the place of the library's entry points."""
import ctypes as C
import importlib.util

import pytest
import torch

from paper_2503_05096_amd import binding, build

OK, ERR_DIM, ERR_HIP = 0, -2, -7
# (name, result type, number of pointer-sized arguments); kv_compact has an int32 among them, which fits
ENTRIES = [("attn_ws", C.c_size_t, 1), ("attn", C.c_int, 11), ("attn_tree", C.c_int, 12), ("accept_ws", C.c_size_t, 1),
           ("accept", C.c_int, 12), ("accept_tree", C.c_int, 14), ("kv_append", C.c_int, 9), ("kv_compact", C.c_int, 10),
           ("commit", C.c_int, 12), ("draft_ws", C.c_size_t, 1), ("draft", C.c_int, 11)]


@pytest.fixture(scope="module")
def module(tmp_path_factory):
    path = build.build_fastcall(out=str(tmp_path_factory.mktemp("fastcall") / "_fastcall.so"), defines=["ADASPEC_FASTCALL_ON_META"])
    spec = importlib.util.spec_from_file_location("_fastcall", path)
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


class Stubs:
    """calls: entry points called so far; status: what they answer; workspace: stands in for binding._workspace"""

    def __init__(self, module):
        self.calls, self.status, self.keep = [], OK, []
        for name, res, n in ENTRIES:
            self.keep.append(C.CFUNCTYPE(res, *[C.c_void_p] * n)(
                (lambda *a: 512) if res is C.c_size_t else (lambda *a, name=name: self.calls.append(name) or self.status)))
        self.workspace = lambda nbytes, device, given, family: torch.empty(nbytes, dtype=torch.uint8, device=device)
        module.setup(tuple(C.cast(f, C.c_void_p).value for f in self.keep), lambda *a: self.workspace(*a), lambda dev: 0, lambda: 0,
                     binding.AdaspecError)


@pytest.fixture
def stubs(module):
    return Stubs(module)


def ints(*shape, dev="meta"):
    return torch.zeros(shape, dtype=torch.int32, device=dev)


def commit_args(next_spec=None, seq=None, seq_lens=None):
    return (ints(3, 4), ints(3), ints(3), ints(3), 3, next_spec, None, None, None, seq, seq_lens, None)


def draft_args(out_rows=None, dev="meta", **kw):
    x = torch.zeros((2, 64), device=dev)
    probs = None if out_rows is None else torch.zeros((5, 64), device=dev)
    return (x, torch.ones(2, device=dev), torch.zeros(2, device=dev), None, probs, out_rows, None, None, None, None)


class Sub(torch.Tensor):
    pass


NOT_PLAIN = {"list": [0, 1, 2], "another device": torch.zeros(3, dtype=torch.int32), "subclass": ints(3).as_subclass(Sub)}


@pytest.mark.parametrize("what", NOT_PLAIN)
def test_optional_arguments_that_are_not_plain_are_left_to_python(module, stubs, what):
    x = NOT_PLAIN[what]
    assert module.commit(*commit_args()) is not NotImplemented and module.draft_sample(*draft_args()) is not NotImplemented
    stubs.calls.clear()
    assert module.commit(*commit_args(next_spec=x)) is NotImplemented
    assert module.commit(*commit_args(seq_lens=x)) is NotImplemented
    assert module.draft_sample(*draft_args(out_rows=x)) is NotImplemented
    assert stubs.calls == []


def test_tensors_without_a_data_pointer_are_left_to_python(module, stubs):
    """Under vmap a tensor has the plain type, but asking for its address throws."""
    seen = []

    def f(x):
        seen.append(module.draft_sample(x, torch.ones(2, device="meta"), torch.zeros(2, device="meta"), None, None, None, None, None,
                                        None, None))
        return x
    torch.vmap(f)(torch.zeros((3, 2, 64), device="meta"))
    assert seen == [NotImplemented] and stubs.calls == []


def every_call(module):
    q, kv, bt = torch.zeros((4, 2, 64), device="meta"), torch.zeros((2, 2, 16, 64), device="meta"), ints(1, 2)
    rows, probs, uni, t = (torch.zeros(n, device="meta") for n in ((4, 64), (3, 64), (4, 2), (1,)))
    attn = (q, kv, kv, bt, ints(1), ints(1), None, 3, 0.0, None, "run", None, None)
    return {"verify_attn": lambda: module.verify_attn(*attn, None),
            "verify_attn_tree": lambda: module.verify_attn(*attn, ints(4)),
            "accept": lambda: module.accept(rows, probs, ints(3), uni, ints(1), t, 3, None, None, None, None, None),
            "accept_tree": lambda: module.accept_tree(rows, probs, ints(3), ints(4), uni, ints(1), t, 3, *[None] * 6),
            "kv_append": lambda: module.kv_append(q, q, kv, kv, bt, ints(1), ints(1), 3, None),
            "kv_compact_path": lambda: module.kv_compact_path(kv, kv, bt, ints(1), ints(1), ints(1, 4), ints(1), 3, None),
            "commit": lambda: module.commit(*commit_args()), "draft_sample": lambda: module.draft_sample(*draft_args())}


def test_statuses_of_the_library(module, stubs):
    """What its checks refuse goes to the Python path; a call that failed in HIP may have enqueued work (commit() would
    append its tokens again): it is made once, and raises."""
    for name, f in every_call(module).items():
        stubs.status = OK
        assert f() is not NotImplemented, name
        stubs.status = ERR_DIM
        assert f() is NotImplemented, name
        stubs.status = ERR_HIP
        stubs.calls.clear()
        with pytest.raises(binding.AdaspecError, match=f"^adaspec_{name}: ") as e:
            f()
        assert e.value.status == ERR_HIP and len(stubs.calls) == 1, name


def test_default_workspaces_when_another_device_is_first_used_meanwhile(module):
    """binding._workspace runs Python, so a thread of another device may make its first call inside it (here: the same
    thread, inside the function that stands in for it)."""
    s, asked = Stubs(module), []

    def on(device, rows):
        module.set_meta_index(device)
        return module.draft_sample(torch.zeros((rows, 64), device="meta"), torch.ones(rows, device="meta"), torch.zeros(rows, device="meta"),
                                   *[None] * 7)

    def workspace(nbytes, device, given, family):
        asked.append(len(asked))
        if len(asked) == 1:
            for other in range(20, 3000, 500):
                assert on(other, 2) is not NotImplemented
            module.set_meta_index(10)
        return torch.empty(1 << 20, dtype=torch.uint8, device="meta")
    s.workspace = workspace
    try:
        assert on(10, 2) is not NotImplemented
        n = len(asked)
        assert n == 7
        assert on(10, 2) is not NotImplemented and on(20, 2) is not NotImplemented
        assert len(asked) == n                            # every device has kept its own
    finally:
        module.set_meta_index(0)


def test_interrupts_inside_a_call_are_not_swallowed(module):
    """Ordinary errors of the Python functions behind the native path send the call to the Python path, which meets them
    again; an interrupt that arrives in one of them ends the call."""
    s = Stubs(module)

    def workspace_raises(e):
        def f(*a):
            raise e
        s.workspace = f
        return module.draft_sample(torch.zeros((2, 64), device="meta"), torch.ones(2, device="meta"), torch.zeros(2, device="meta"),
                                   *[None] * 7)

    class Stream:
        def __init__(self, e):
            self.e = e

        @property
        def cuda_stream(self):
            raise self.e
    module.set_meta_index(4000)                           # a device without a workspace yet
    try:
        assert workspace_raises(RuntimeError("out of memory")) is NotImplemented
        with pytest.raises(KeyboardInterrupt):
            workspace_raises(KeyboardInterrupt())
    finally:
        module.set_meta_index(0)
    assert module.commit(*commit_args()[:-1], Stream(ValueError())) is NotImplemented
    with pytest.raises(SystemExit):
        module.commit(*commit_args()[:-1], Stream(SystemExit()))
    assert s.calls == []


@pytest.mark.parametrize("what", ["missing", "another torch"])
def test_the_binding_without_its_native_path(what, monkeypatch):
    """The Python route is complete: without the module (or with one built for another torch) the binding warns once and
    takes it."""
    import paper_2503_05096_amd as pkg
    import sys
    import types
    name = "paper_2503_05096_amd._fastcall"
    monkeypatch.setattr(binding, "_fast", None)
    monkeypatch.delattr(pkg, "_fastcall", raising=False)
    monkeypatch.setitem(sys.modules, name, None if what == "missing" else types.SimpleNamespace(torch_version="0.0"))
    t = torch.zeros(2, 2)
    with pytest.warns(RuntimeWarning, match="no native call path"):
        with pytest.raises(AssertionError):               # the Python route's own check: not on a GPU
            pkg.commit(ints(1, 1, dev="cpu"), ints(1, dev="cpu"), ints(1, dev="cpu"), ints(1, dev="cpu"), max_spec_len=0)
    fast = binding._fast
    for f, n in (("verify_attn", 14), ("accept", 12), ("accept_tree", 14), ("kv_append", 9), ("kv_compact_path", 9), ("commit", 12),
                 ("draft_sample", 10)):
        assert getattr(fast, f)(*[t] * n) is NotImplemented


def test_a_library_without_the_native_path_can_be_built(tmp_path, monkeypatch, capsys):
    """A machine without a host C++ compiler still gets the library; no older module stays beside it."""
    stale = tmp_path / "_fastcall.so"
    stale.write_bytes(b"")
    monkeypatch.setenv("CXX", str(tmp_path / "no-compiler"))
    monkeypatch.setattr(build, "FASTCALL_PATH", str(stale))
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "BUILD_DIR", str(tmp_path / "objects"))
    monkeypatch.setattr(build, "HIPCC", "true")
    build.build_library()
    assert not stale.exists() and "_fastcall.so was not built" in capsys.readouterr().err
