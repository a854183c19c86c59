"""The native binding of the hot calls takes the ordinary call, and leaves every other one to the Python binding, with the same outcome."""
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HP = (1e-3, 0.9, 0.95, 1e-8, 0.1, 3)


class Sub(torch.Tensor):
    pass


def _state(dtype):
    T, d, F, V = 33, 64, 128, 50
    s = inputs.layer_inputs(inputs.StemShape("bind", d, F, V, 1, T, dtype), 3, device=DEV)
    dt = s["x"].dtype
    new = lambda *n, t=dt: torch.zeros(*n, dtype=t, device=DEV)
    i32, f32 = torch.int32, torch.float32
    s.update(ctx=Hn.make_ctx(inputs.StemShape("bind", d, F, V, 1, T, dtype), T), y=new(T, d), G=new(T, F), H=new(T, F), dx=new(T, d),
             dU=new(T, F), dWg=new(F, d, t=f32), dWd=new(d, F, t=f32), si=new(T, t=i32), pe=new(T, t=i32), ui=new(T, t=i32),
             so=new(T + 1, t=i32), nu=new(1, t=i32), dE=new(T, F, t=f32), m=new(V, F, t=f32), v=new(V, F, t=f32),
             ma=s["E"].float() if dtype == "bf16" else None)
    return s


def _step(s):
    """The calls of a training step and a residual forward, as (native function, its arguments, the call)."""
    g = s.__getitem__
    yield "ffn_forward", [*map(g, ("ctx", "x", "ids", "W_gate", "W_down", "E", "y", "G", "H")), None, None, None, None], \
        lambda: L.stem_ffn_forward(*map(g, ("ctx", "x", "ids", "W_gate", "W_down", "E", "y", "G", "H")))
    names = ("ctx", "dy", "x", "ids", "W_gate", "W_down", "E", "G", "H", "dx", "dWg", "dWd", "dU")
    yield "ffn_backward", [*map(g, names), False, None, None, None], lambda: L.stem_ffn_backward(*map(g, names))
    names_e = ("ctx", "ids", "dU", "si", "pe", "ui", "so", "nu", "dE")
    yield "embed_grad", [*map(g, names_e), None, None], lambda: L.stem_embed_grad(*map(g, names_e))
    names_p = ("ctx", "dU", "pe", "so", "dE")
    yield "embed_grad_presorted", [*map(g, names_p), None, None], lambda: L.stem_embed_grad_presorted(*map(g, names_p))
    names_a = ("ctx", "ui", "nu", "dE", "E", "ma", "m", "v")
    yield "embed_sparse_adamw", [*map(g, names_a), *HP, None, None], lambda: L.stem_embed_sparse_adamw(*map(g, names_a), *HP)
    if s["y"].dtype == torch.bfloat16:
        names_r = ("ctx", "x", "ids", "W_gate", "W_down", "E", "x", "y")
        yield "ffn_forward_residual", [*map(g, names_r), None, None, None], lambda: L.stem_ffn_forward_residual(*map(g, names_r))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_both_bindings_make_the_same_calls(dtype, monkeypatch):
    native = L._bind or L._load_bind()
    a, b = _state(dtype), _state(dtype)
    for name, args, _ in _step(a):
        assert getattr(native, name)(*args) == L.STEM_OK, name     # the ordinary call is made here

    class No:
        def __getattr__(self, name):
            return lambda *args: None
    monkeypatch.setattr(L, "_bind", No())
    for _, _, call in _step(b):
        call()
    L.stem_sync_status(a["ctx"])
    L.stem_sync_status(b["ctx"])
    for k, t in a.items():
        if isinstance(t, torch.Tensor):
            assert torch.equal(t, b[k]), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_lazily_cloned_tensors_are_written_apart_from_their_source(dtype):
    native = L._bind or L._load_bind()
    a, b = _state(dtype), _state(dtype)
    source = {k: t for k, t in b.items() if isinstance(t, torch.Tensor)}
    before = {k: t.clone() for k, t in source.items()}
    b.update({k: torch._lazy_clone(t) for k, t in source.items()})
    for (name, args, _), (_, lazy, _) in zip(_step(a), _step(b)):
        assert getattr(native, name)(*args) == getattr(native, name)(*lazy) == L.STEM_OK, name
    if dtype == "bf16":   # in place
        x = a["x"].clone()
        shared = torch._lazy_clone(x)
        L.stem_ffn_forward_residual(b["ctx"], shared, *[b[k] for k in ("ids", "W_gate", "W_down", "E")], shared, shared)
        want = torch.empty_like(x)
        L.stem_ffn_forward_residual(b["ctx"], x, *[b[k] for k in ("ids", "W_gate", "W_down", "E")], x, want)
        assert torch.equal(shared, want) and torch.equal(x, a["x"])
    L.stem_sync_status(a["ctx"])
    L.stem_sync_status(b["ctx"])
    for k, t in source.items():
        assert torch.equal(t, before[k]), k          # nothing was written through it
        assert torch.equal(a[k], b[k]), k


def test_what_is_not_ordinary_is_left_to_the_other_binding():
    native = L._bind or L._load_bind()
    s = _state("bf16")
    args = dict(zip(("ctx", "x", "ids", "W_gate", "W_down", "E", "y", "G", "H", "event", "stream", "E_rows", "T"), next(_step(s))[1]))
    call = lambda **o: native.ffn_forward(*{**args, **o}.values())
    T, d = s["x"].shape
    assert call() == L.STEM_OK and call(stream=torch.cuda.current_stream()) == L.STEM_OK and call(T=T - 1, E_rows=50) == L.STEM_OK
    assert call(T=T + 1) == L.STEM_ERR_SHAPE and call(y=None) == L.STEM_ERR_INVALID_ARG
    wrong = [dict(x=s["x"].float()), dict(x=s["x"].cpu()), dict(x=torch.zeros(d, T, dtype=torch.bfloat16, device=DEV).t()),
             dict(x=s["x"].as_subclass(Sub)), dict(x=s["x"].to("meta")), dict(ids=s["ids"].long()), dict(x=3), dict(T=1.0), dict(T=1 << 70),
             dict(stream="s"), dict(event=1.5), dict(ctx=3), dict(E=None)]
    for o in wrong:
        assert call(**o) is None, o
    L.stem_sync_status(s["ctx"])
    # and there a subclass is taken, and the others named
    L.stem_ffn_forward(s["ctx"], s["x"].as_subclass(Sub), s["ids"], s["W_gate"], s["W_down"], s["E"], s["y"])
    for kw, error in ((dict(x=s["x"].float()), TypeError), (dict(x=s["x"].cpu()), ValueError), (wrong[2], ValueError), (dict(ids=s["ids"].long()), TypeError)):
        with pytest.raises(error, match=next(iter(kw))):
            L.stem_ffn_forward(s["ctx"], *{**{k: s[k] for k in ("x", "ids", "W_gate", "W_down", "E", "y")}, **kw}.values())
    L.stem_sync_status(s["ctx"])
    s["ctx"].close()
    assert call() is None
    with pytest.raises(L.StemError):
        L.stem_ffn_forward(s["ctx"], s["x"], s["ids"], s["W_gate"], s["W_down"], s["E"], s["y"])
