"""The native way of the calls that are given all their buffers (csrc/calls.cpp): the same results as the general way, which
allocates them, on the current stream, and the same refusals."""
import ctypes

import pytest
import torch

from paper_2411_09909_amd import binding

pytestmark = pytest.mark.gpu

FMT = binding.make_format(binding.FP8_E5M2, True, 32)


def randn(*shape, seed=0):
    return torch.randn(shape, generator=torch.Generator("cuda").manual_seed(seed), device="cuda").to(torch.bfloat16)


def like(pair):
    return {"codes": torch.zeros_like(pair[0]), "scales": torch.zeros_like(pair[1])}


def same(a, b):
    a, b = (t if isinstance(t, tuple) else (t,) for t in (a, b))
    return all(torch.equal(p, q) for p, q in zip(a, b))


def taken(monkeypatch, name):
    """Counts the calls of the native function `name` that it took."""
    binding.load()
    class Spy:
        count = 0
        def __getattr__(self, attr):
            def call(*args):
                rc = getattr(calls, attr)(*args)
                Spy.count += attr == name and rc is not None
                return rc
            return call
    calls = binding._calls
    monkeypatch.setattr(binding, "_calls", Spy())
    return Spy


@pytest.mark.parametrize("k_axis", [-1, 0])
@pytest.mark.parametrize("scaled", [False, True])
def test_casts(monkeypatch, k_axis, scaled):
    x = randn(64, 96)
    pair = binding.tensor_scale(x) if scaled else None
    want = binding.quantize(FMT, x, k_axis=k_axis, tensor_pair=pair)
    wantb = binding.quantize_batched(FMT, x[None], k_axis=1 if k_axis == 0 else -1)
    spy, out = taken(monkeypatch, "quantize"), like(want)
    assert same(binding.quantize(FMT, x, k_axis=k_axis, tensor_pair=pair, **out), want) and spy.count == 1
    spy, out = taken(monkeypatch, "quantize_batched"), like(wantb)
    assert same(binding.quantize_batched(FMT, x[None], k_axis=1 if k_axis == 0 else -1, **out), wantb) and spy.count == 1
    spy, two = taken(monkeypatch, "tensor_scale"), torch.zeros(2, device="cuda")
    assert same(binding.tensor_scale(x, out=two), binding.tensor_scale(x)) and spy.count == 1


@pytest.mark.parametrize("kind", ["plain", "batched", "scaled", "prepared", "window of a wider C"])
def test_products(monkeypatch, kind):
    M, N, K = 40, 96, 256
    a, b = randn(M, K, seed=1), randn(N, K, seed=2)
    pairs = {}
    if kind == "scaled":
        pairs = {"a_pair": binding.tensor_scale(a), "b_pair": binding.tensor_scale(b)}
    qa, qb = (binding.quantize(FMT, t, tensor_pair=p) for t, p in zip((a, b), pairs.values() or (None, None)))
    if kind == "batched":
        qa, qb = ([torch.stack([t, t]) for t in q] for q in (qa, qb))
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    if kind == "prepared":
        prepared = binding.prepare_weights(FMT, *qb)
        call, name = lambda **kw: binding.gemm_prepared(FMT, *qa, *qb, prepared, **kw), "gemm_prepared"
    else:
        call, name = lambda **kw: binding.gemm(FMT, *qa, *qb, **pairs, **kw), "gemm"
    want = call()
    wide = torch.zeros(want.shape[:-1] + (N + 32,), device="cuda")
    out = wide[..., :N] if kind == "window of a wider C" else torch.zeros_like(want)
    spy = taken(monkeypatch, name)
    assert same(call(out=out, workspace=ws), want) and spy.count == 1 and not wide[..., N:].any()


@pytest.mark.parametrize("merged", [False, True])
def test_attention(monkeypatch, merged):
    q, k, v = randn(4, 64, 64, seed=3), randn(2, 96, 64, seed=4), randn(2, 96, 64, seed=5)
    ops = [t for x, axis in ((q, -1), (k, -1), (v, 1)) for t in binding.quantize_batched(FMT, x, k_axis=axis)]
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    want = binding.attention(FMT, *ops, 0.125, True, merged=merged)
    spy = taken(monkeypatch, "attention")
    assert same(binding.attention(FMT, *ops, 0.125, True, out=torch.zeros_like(want), workspace=ws, merged=merged), want) and spy.count == 1
    one = [t for t in binding.quantize_batched(FMT, q[:, :1].contiguous())] + ops[2:]
    want = binding.attention_decode(FMT, *one, 0.125, True, key_splits=2)
    spy = taken(monkeypatch, "attention_decode")
    got = binding.attention_decode(FMT, *one, 0.125, True, key_splits=2, out=torch.zeros_like(want), workspace=ws)
    assert same(got, want) and spy.count == 1


def test_runs_on_the_current_stream():
    x, side = randn(4096, 4096), torch.cuda.Stream()
    want = binding.quantize(FMT, x)
    out = like(want)
    late = torch.zeros_like(x)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):
            late.copy_(x.neg())
        late.copy_(x)
        got = binding.quantize(FMT, late, **out)
    side.synchronize()
    assert same(got, want)


def test_refusals_stay():
    x = randn(64, 96)
    q = binding.quantize(FMT, x)
    out, ws = torch.empty(64, 64, device="cuda"), torch.empty(0, dtype=torch.uint8, device="cuda")
    with pytest.raises(binding.AmxError, match="device memory only"):
        binding.quantize(FMT, x.cpu(), **like(q))
    with pytest.raises(AssertionError):
        binding.quantize(FMT, x[None], **like(q))
    with pytest.raises(binding.AmxError, match="unsupported strides"):
        binding.quantize(FMT, x[:, ::3], **like(q))
    with pytest.raises(AssertionError):
        binding.gemm(FMT, q[0][:, ::2], q[1], *q, out=out, workspace=ws)
    with pytest.raises(binding.AmxError, match="both tensor-scale pairs"):
        binding.gemm(FMT, *q, *q, out=out, workspace=ws, a_pair=torch.ones(2, device="cuda"))
    with pytest.raises(binding.AmxError, match="workspace of [0-9]+ bytes needed, 0 given"):
        binding.gemm(FMT, *q, *q, out=out, workspace=ws)


@pytest.mark.parametrize("other", [bytes(FMT), binding.gemm_options(e5m2_kernel=32, tile=2, few_rows=1)], ids=["bytes", "options"])
def test_only_a_format_is_a_format(other):
    """Four 32-bit numbers, the same bytes as a format's (both of these would be valid ones), are refused like any other type."""
    assert bytes(other) == bytes(FMT)
    x = randn(64, 96)
    q = binding.quantize(FMT, x)
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    with pytest.raises(AttributeError):
        binding.quantize(other, x, **like(q))
    with pytest.raises(AttributeError):
        binding.quantize_batched(other, x[None], codes=q[0][None], scales=q[1][None])
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        binding.gemm(other, *q, *q, out=torch.empty(64, 64, device="cuda"), workspace=ws)
    derived = type("Derived", (binding.AmxFormat,), {})(*(getattr(FMT, name) for name, _ in FMT._fields_))
    out = like(q)
    assert same(binding.quantize(derived, x, **out), q)
