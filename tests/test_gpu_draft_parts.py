"""Draft sampling in row parts (csrc/draft_parts.hip) over all pairs of storage types: vocabularies around a step of 256
chunks, a wavefront's share, a part, and the largest one, on the path AUTO takes for them; rows with few finite logits, the
ends of the uniforms' range, scattered rows. Bar of the other draft tests (one ulp per stored probability, tokens equal or
a counted near-tie)."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_draft import _check, pkg  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

T = np.array([1.0, 0.0, 0.5, 1.3], np.float32)
U = np.array([0.0, 0.5, 1.0 - 2.0 ** -24, 0.37], np.float32)


def _logits(R, V, ldt, seed=3, masked=0.0):
    rng = np.random.default_rng(seed + V)
    x = (2.5 * rng.standard_normal((R, V))).astype(np.float32)
    if masked:
        gone = rng.random((R, V)) < masked
        gone[np.arange(R), rng.integers(0, V, R)] = False
        x[gone] = -np.inf
    return x if ldt == "f32" else W.f32_to_bf16_bits(x) if ldt == "bf16" else x.astype(np.float16)


@pytest.mark.parametrize("V", [32768, 32776, 49160, 50184])
@pytest.mark.parametrize("ldt,pdt", [(a, b) for a in ("f32", "f16", "bf16") for b in ("f32", "f16", "bf16")])
def test_draft_parts_types(ldt, pdt, V, oracle_mod, pkg):  # noqa: F811
    _check(_logits(4, V, ldt), ldt, pdt, T, U, oracle_mod, pkg)


@pytest.mark.parametrize("V,ldt,pdt", [(128256, "f32", "bf16"), (131080, "bf16", "bf16"), (262144, "f16", "f32"),
                                       (524288, "f32", "f32"), (524280, "bf16", "bf16")])
def test_draft_parts_large_vocabularies(V, ldt, pdt, oracle_mod, pkg):  # noqa: F811
    _check(_logits(3, V, ldt), ldt, pdt, T[:3], U[:3], oracle_mod, pkg)


@pytest.mark.parametrize("V", [8, 8192, 8200, 16384 + 8, 40000])
def test_draft_parts_forced_on_small_rows(V, oracle_mod, pkg):  # noqa: F811
    _check(_logits(4, V, "bf16"), "bf16", "bf16", T, U, oracle_mod, pkg, path="split")


def test_draft_parts_masked_rows_and_scattered_output(oracle_mod, pkg):  # noqa: F811
    rows = np.array([5, 0, 6, 2], np.int32)
    for ldt in ("f32", "bf16"):
        _check(_logits(4, 50000, ldt, masked=0.999), ldt, ldt, T, U, oracle_mod, pkg, out_rows=rows, n_prob_rows=7)


@pytest.mark.parametrize("V", [32768, 50272, 128256, 262144])
@pytest.mark.parametrize("ldt", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("T", [1.0, 0.3, 0.02])
def test_draft_rows_in_fp32_sum_to_one(V, ldt, T, pkg):  # noqa: F811
    """What every probability of a row is off by in common: reciprocal of the normaliser 6e-8, fp32 sums of up to 512 terms per
    thread in it 1.5e-7, the exponential's rounding, which the few largest weights share, 1.2e-7: 3.3e-7."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(V)
    x = (3.0 * torch.randn((64, V), generator=gen, device="cuda")).to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[ldt])
    probs, _, _ = pkg.draft_sample(x, torch.full((64,), T, device="cuda"), torch.rand(64, generator=gen, device="cuda"),
                                   probs_dtype=torch.float32)
    torch.cuda.synchronize()
    assert float((probs.double().sum(1) - 1.0).abs().max()) <= 3.3e-7


@pytest.mark.parametrize("V", [50184, 262144])
@pytest.mark.parametrize("ldt", ["bf16", "f16", "f32"])
def test_draft_parts_at_temperatures_next_to_zero(V, ldt, oracle_mod, pkg):  # noqa: F811
    _check(_logits(4, V, ldt), ldt, ldt, np.array([1e-8, 1e-10, 1e-7, 1e-9], np.float32), U, oracle_mod, pkg)


def test_draft_parts_greedy_rows_with_rising_and_equal_maxima(oracle_mod, pkg):  # noqa: F811
    """The arg-max is searched for only where a chunk raises the running maximum: rows that rise to the last element, fall
    from the first, repeat their maximum in later elements, chunks, steps and parts, or hold one finite logit."""
    V = 50184
    x = np.zeros((5, V), np.float32)
    # (63 steps: the smallest probability, e^-63 / 800 = 6e-31, is a normal number of fp32 and bf16; the exponential of what
    # is not comes out as 0, which the oracle's comparison of fp32 rows does not allow)
    x[0] = np.floor(np.arange(V) / 800.0)                            # ends on a run of equal maxima
    x[1] = -np.floor(np.arange(V) / 800.0)
    x[2, [3, 5, 11, 2048, 4096 * 8, V - 1]] = 7.0                    # the lowest of them
    x[3] = -np.inf
    x[3, V - 1] = -30.0
    x[4, :] = -2.0
    T5, U5 = np.zeros(5, np.float32), np.full(5, 0.5, np.float32)
    for ldt in ("bf16", "f16", "f32"):
        y = x if ldt == "f32" else W.f32_to_bf16_bits(x) if ldt == "bf16" else x.astype(np.float16)
        _check(y, ldt, ldt, T5, U5, oracle_mod, pkg)


@pytest.mark.parametrize("V", [16384, 32768, 50184, 128256])
@pytest.mark.parametrize("ldt", ["bf16", "f16", "f32"])
def test_draft_rows_with_a_nan(V, ldt, pkg):  # noqa: F811
    """A NaN among the logits makes its whole row NaN: token 0 and confidence 0, or the arg-max of the rest for a greedy row.
    NaNs of both signs, beside finite logits of their thread and beside nothing but masked ones; the other rows stay as they are."""
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[ldt]
    gen = torch.Generator(device="cuda").manual_seed(V)
    R = 12
    x = 3.0 * torch.randn((R, V), generator=gen, device="cuda")
    x[4:8, 2048:V - 2048] = -float("inf")                            # (rows 4-7: threads whose other logits are all masked)
    x = x.to(dt)
    t = torch.tensor([0.8, 0.0, 1.0, 0.0], device="cuda").repeat(3)
    u = torch.rand(R, generator=gen, device="cuda")
    rest = x.float().clone()
    clean = [v.clone() for v in pkg.draft_sample(x, t, u)]
    bits = x.view(torch.int32 if ldt == "f32" else torch.int16)
    plus, minus = (0x7fffffff, -1) if ldt == "f32" else (0x7fff, -1)
    for r, (i, pattern) in enumerate([(5, plus), (V // 2 + 3, plus), (V - 1, minus), (V // 3, minus)] * 2):
        bits[r, i] = pattern
        rest[r, i] = -float("inf")
    # beside the largest logit of its row
    bits[1, (int(rest[1].argmax()) & ~7) + (0 if int(rest[1].argmax()) & 7 else 1)] = plus
    q, tok, conf = pkg.draft_sample(x, t, u)
    torch.cuda.synchronize()
    for r in range(R):
        if r >= 8:
            assert torch.equal(q[r], clean[0][r]) and tok[r] == clean[1][r] and conf[r] == clean[2][r]
            continue
        assert bool(torch.isnan(q[r]).all()), (r, int(torch.isnan(q[r]).sum()))
        if float(t[r]) > 0:
            assert int(tok[r]) == 0 and float(conf[r]) == 0.0
        else:
            assert int(tok[r]) == int(rest[r].argmax()) and bool(torch.isnan(conf[r]))


@pytest.mark.parametrize("V,ldt", [(16384, "bf16"), (16392, "f32"), (32768, "f16"), (131072, "bf16")])
def test_draft_rows_at_an_infinite_temperature(V, ldt, pkg):  # noqa: F811
    """T = inf: every token equally likely, whatever the finite logits."""
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[ldt]
    gen = torch.Generator(device="cuda").manual_seed(V)
    x = (3.0 * torch.randn((4, V), generator=gen, device="cuda")).to(dt)
    u = torch.tensor([0.0, 0.25, 0.5, 1.0 - 2.0 ** -24], device="cuda")
    q, tok, conf = pkg.draft_sample(x, torch.tensor([float("inf"), float("inf"), 3e38, float("inf")], device="cuda"), u)
    torch.cuda.synchronize()
    want = torch.tensor(1.0 / V, device="cuda").to(dt).float()
    assert bool(((q.float() - want).abs() <= {"f32": 2.0 ** -22, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[ldt] * want + (6e-8 if ldt == "f16" else 0.0)).all())
    assert bool(((tok.double() - u.double() * V).abs() <= 1e-5 * V + 1).all()) and bool((conf > 0).all())


# whole rows, rows in parts (threads of both sizes, all pairs of equal element size), a last part that is nearly empty, the most parts
@pytest.mark.parametrize("R,V,dtype", [(4, 16384, "bfloat16"), (6, 32776, "bfloat16"), (5, 50184, "float32"), (70, 65544, "float16"),
                                       (128, 128256, "bfloat16"), (3, 524288, "float32")])
@pytest.mark.parametrize("mapped,path", [(False, "auto"), (False, "split"), (True, "auto")])
def test_draft_rows_in_place(R, V, dtype, mapped, path, pkg):  # noqa: F811
    """The probabilities may go where the logits are, row by row: the same result as beside them on the path that takes them."""
    import torch
    if path == "split" and dtype == "float32":
        pytest.skip("the split form takes fp32 rows by itself only")
    beside = path if path == "split" or mapped else "fast" if dtype != "float32" and V > 24576 else "vector"
    gen = torch.Generator(device="cuda").manual_seed(R + V)
    x = 3.0 * torch.randn((R, V), generator=gen, device="cuda")
    x[::3, :V // 2] = -float("inf")
    x[1, 77] = float("nan")
    x = x.to(getattr(torch, dtype))
    t = torch.tensor([0.8, 1.0, 0.0, 1.3], device="cuda").repeat(R)[:R]
    u = torch.rand(R, generator=gen, device="cuda")
    want = [v.clone() for v in pkg.draft_sample(x, t, u, path=beside)]
    buffer = torch.zeros((R + 3, V), dtype=x.dtype, device="cuda")
    first = 2 if mapped else 0
    buffer[first:first + R] = x
    rows = torch.arange(first, first + R, dtype=torch.int32, device="cuda") if mapped else None
    logits = buffer[first:first + R]
    _, tok, conf = pkg.draft_sample(logits, t, u, draft_probs=buffer if mapped else logits, out_rows=rows, path=path)
    torch.cuda.synchronize()
    assert torch.equal(tok, want[1]) and torch.equal(conf.nan_to_num(-1.0), want[2].nan_to_num(-1.0))
    assert torch.equal(logits.float().nan_to_num(-1.0), want[0].float().nan_to_num(-1.0))
    assert bool((buffer[:first] == 0).all()) and bool((buffer[first + R:] == 0).all())


@pytest.mark.parametrize("V", [8192, 16384, 32768, 50184, 128256])
@pytest.mark.parametrize("ldt,path", [("bf16", "auto"), ("bf16", "split"), ("bf16", "fast"), ("bf16", "vector"), ("f16", "auto"), ("f32", "auto")])
def test_draft_rows_masked_with_the_lowest_number(V, ldt, path, oracle_mod, pkg):  # noqa: F811
    """Masked by the type's lowest number in place of -inf, alone and in stretches (threads, parts of which nothing else is left): a
    product of it with log2(e) / T overflows for bf16."""
    x = _logits(4, V, "f32", seed=8, masked=0.3)
    x[:, V // 4:V // 2] = -np.inf
    x[:, V - 256:] = -np.inf
    x[0, V // 2 + 5] = 3.0                                        # (every row has something left)
    gone = np.isneginf(x)
    y = x if ldt == "f32" else W.f32_to_bf16_bits(x) if ldt == "bf16" else x.astype(np.float16)
    y[gone] = {"f32": np.finfo(np.float32).min, "f16": np.finfo(np.float16).min, "bf16": np.uint16(0xFF7F)}[ldt]
    _check(y, ldt, ldt, T, U, oracle_mod, pkg, path=path)
    if ldt == "bf16" or path == "auto":                           # far from T = 1 the product is finite, but coarse
        _check(y, ldt, ldt, np.array([100.0, 30.0, 3.0, 300.0], np.float32), U, oracle_mod, pkg, path=path)
    if ldt == "f16":
        _check(y, ldt, ldt, np.array([1e-5, 1e-6, 1e-7, 1e-8], np.float32), U, oracle_mod, pkg, path=path)
