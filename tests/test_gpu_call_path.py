"""The C++ call path of the plain entry points against the marshalled calls of the
same arguments: the same bits with and without outputs given, on the current stream
whichever it is, and the same errors and results for what it declines."""
import pytest
import torch

import paper_2603_04427_amd as tk
from gpu_cases import device, say
from paper_2603_04427_amd import binding

pytestmark = pytest.mark.gpu


def _inputs(dtype=torch.bfloat16, b=2, hq=4, hkv=2, sq=33, sk=65, r=32, dv=64):
    g = torch.Generator(device="cuda").manual_seed(5)
    mk = lambda *s: torch.randn(*s, generator=g, device=device(), dtype=dtype)  # noqa: E731
    return mk(b, hq, sq, r), mk(b, hkv, sk, r), mk(b, hkv, sk, dv)


def _same(a, b):
    a, b = (a, b) if isinstance(a, tuple) else ((a,), (b,))
    assert len(a) == len(b) and all(torch.equal(x, y) and x.dtype == y.dtype for x, y in zip(a, b))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("own_stream", [False, True])
def test_attention_calls_match_the_marshalled_ones(causal, own_stream):
    say(f"call path causal={causal} own_stream={own_stream}")
    q, k, v = _inputs()
    q32, k32, v32 = _inputs(torch.float32)
    do = torch.randn_like(q[..., :1]).expand(2, 4, 33, 64).contiguous()
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if own_stream else torch.cuda.current_stream()):
        assert binding._native("prefill", q, k, v, None, causal, 0.0, None) is not None
        _same(tk.tk_attn_prefill(q, k, v, causal=causal), tk.prepare_prefill(q, k, v, causal=causal)())
        _same(tk.tk_attn_prefill(q32, k32, v32, causal=causal, scale=0.3),
              tk.prepare_prefill(q32, k32, v32, causal=causal, scale=0.3)())
        o, lse = tk.tk_attn_prefill_lse(q, k, v, causal=causal)
        _same((o, lse), tk.prepare_prefill_lse(q, k, v, causal=causal)())
        want = tk.prepare_prefill_backward(q, k, v, o, do, lse, causal)()
        _same(tk.tk_attn_prefill_backward(q, k, v, o, do, lse, causal), want)
        given = torch.full_like(o, 7.0), torch.full_like(lse, 7.0)
        out = tk.tk_attn_prefill_lse(q, k, v, *given, causal=causal)
        assert out[0] is given[0] and out[1] is given[1]
        _same(out, (o, lse))
        dk = torch.full_like(k, 7.0)
        out = tk.tk_attn_prefill_backward(q, k, v, o, do, lse, causal, dK=dk)
        assert out[1] is dk
        _same(out, want)
        torch.cuda.synchronize()


@pytest.mark.parametrize("keys", ["bf16", "fp8", "int4"])
@pytest.mark.parametrize("paged", [False, True])
def test_projection_and_append_match_the_marshalled_ones(keys, paged):
    say(f"call path append {keys} paged={paged}")
    dev = device()
    x, w = torch.randn(2, 5, 64, device=dev).bfloat16(), torch.randn(2 * 32, 64, device=dev).bfloat16()
    y = torch.full((2, 2, 5, 32), 7.0, device=dev, dtype=torch.bfloat16)
    _same(tk.tk_project_heads(x, w, 2), tk.prepare_project_heads(x, w, 2)())
    assert tk.tk_project_heads(x, w, 2, y) is y
    _same(y, tk.prepare_project_heads(x, w, 2)())
    vn = torch.randn(2, 2, 5, 64, device=dev).bfloat16()
    pos = torch.tensor([0, 60], dtype=torch.int32, device=dev)
    lead = (4, 2, 64) if paged else (2, 2, 128)
    table = torch.tensor([[3, 1], [0, 2]], dtype=torch.int32, device=dev) if paged else None
    caches = []
    for call in (tk.tk_cache_append, lambda *a, **kw: tk.prepare_cache_append(*a, **kw)()):
        kc = torch.zeros(*lead, 16 if keys == "int4" else 32, device=dev,
                         dtype=torch.bfloat16 if keys == "bf16" else torch.uint8)
        vc = torch.zeros(*lead, 64, device=dev, dtype=torch.bfloat16)
        ks = None if keys == "bf16" else torch.zeros(*lead, device=dev)
        call(y, vn, pos, kc, vc, k_scale=ks, block_table=table, block_size=64 if paged else 0)
        caches.append(tuple(t for t in (kc, vc, ks) if t is not None))
    _same(*caches)


def test_declined_calls_are_marshalled_and_refused_as_before():
    q, k, v = _inputs()
    want = tk.prepare_prefill(q, k, v)()

    class Sub(torch.Tensor):
        pass

    for args in ((q.as_subclass(Sub), k, v, None, True, 0.0, None), (q, k, v, None, 1, 0.0, None),
                 (q, k, v, None, True, 0, None), (q, k, v, None, True, 0.0, torch.cuda.current_stream())):
        assert binding._native("prefill", *args) is None
        _same(tk.tk_attn_prefill(*args).as_subclass(torch.Tensor), want)
    with pytest.raises(ValueError, match="contiguous"):
        tk.tk_attn_prefill(q.transpose(1, 2), k, v)
    with pytest.raises(TypeError, match="dtype"):
        tk.tk_attn_prefill(q, k.float(), v)
    with pytest.raises(ValueError, match="GPU"):
        tk.tk_attn_prefill(q.cpu(), k, v)
    with pytest.raises(ValueError, match="mismatch"):
        tk.tk_attn_prefill(q, k[:, :1].contiguous(), v)
    with pytest.raises(ValueError, match="wrong shape"):
        tk.tk_attn_prefill(q, k, v, torch.empty_like(q))
    with pytest.raises(tk.TkError) as e:
        tk.tk_attn_prefill(*_inputs(r=48))
    assert e.value.status == binding.TK_ERR_UNSUPPORTED and "tk_attn_prefill" in str(e.value)
    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    with Mode():
        _same(tk.tk_attn_prefill(q, k, v), want)
    assert torch.empty in seen
