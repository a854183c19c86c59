"""Weight gradients that share a launch, against the oracle, on every tiling and K split; and where they may not share one."""
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(T, d, F, up, accumulate=False):
    V = 300
    s = inputs.StemShape("dw", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=71, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T, reserve=L.STEM_RESERVE_UP if up else 0)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    ids = inp["ids"].cpu().numpy()
    e = lambda *sh, dt=torch.bfloat16: torch.empty(*sh, dtype=dt, device=DEV)  # noqa: E731
    y, G, Up, H, dx, dU = e(T, d), e(T, F), e(T, F), e(T, F), e(T, d), e(T, F)
    start = 0.5 if accumulate else float("nan")
    dWg, dWu = (torch.full((F, d), start, device=DEV) for _ in range(2))
    dWd = torch.full((d, F), start, device=DEV)
    a = (ctx, inp["x"], inp["ids"], inp["W_gate"])
    if up:
        Wu = inputs.normal((F, d), 0.02, 72, torch.bfloat16, DEV)
        L.stem_ffn_up_forward(*a, Wu, inp["W_down"], inp["E"], y, G, Up, H)
        L.stem_ffn_up_backward(ctx, inp["dy"], *a[1:], Wu, inp["W_down"], inp["E"], G, Up, H, dx, dWg, dWu, dWd, dU,
                               accumulate=accumulate)
        bw = O.up_backward(f64["dy"], f64["x"], ids, f64["W_gate"], inputs.to_f64(Wu), f64["W_down"], f64["E"])
    else:
        L.stem_ffn_forward(*a, inp["W_down"], inp["E"], y, G, H)
        L.stem_ffn_backward(ctx, inp["dy"], *a[1:], inp["W_down"], inp["E"], G, H, dx, dWg, dWd, dU, accumulate=accumulate)
        bw = O.ffn_backward(f64["dy"], f64["x"], ids, f64["W_gate"], f64["W_down"], f64["E"])
    L.stem_sync_status(ctx)
    out = {"dW_gate": dWg, "dW_down": dWd, "dx": dx, **({"dW_up": dWu} if up else {})}
    off = 0.5 if accumulate else 0.0
    errs = {k: Hn.max_rel(v.float().cpu(), bw[k] + (off if k != "dx" else 0.0)) for k, v in out.items()}
    assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
    ctx.close()


@pytest.mark.parametrize("T,d,F,up,route", [
    (700, 192, 576, False, (1, 128, 128, 1)),        # ragged in M, N and K
    (1100, 128, 320, False, (1, 128, 128, 4)),       # K slices, the last shorter; tiles of one product end inside an XCD's run
    (1100, 128, 320, True, (1, 128, 128, 4)),
    (2500, 704, 2816, False, (1, 256, 128, 1)),
    (2500, 704, 2816, True, (1, 256, 128, 1)),
    (9000, 512, 2112, False, (1, 256, 128, 2)),      # slices of 256x128 tiles
    (2001, 1088, 4032, False, (1, 256, 256, 1)),
    (2001, 1088, 4032, True, (1, 256, 256, 1)),      # 3 x 80 tiles
    (7575, 192, 2112, False, (1, 256, 128, 4)),
    (2218, 128, 384, False, (1, 128, 128, 7)),       # a slice count that does not divide the K tiles
    (1999, 2048, 8192, False, (1, 256, 256, 1)),     # whole rounds either way
    (613, 1344, 5824, False, (0,)),                  # a launch each
])
def test_weight_gradients_in_one_launch(T, d, F, up, route):
    ws = min(64 << 20, 32 * d * max(T, F))
    assert Hn.route_weight_grads(T, d, F, 3 if up else 2, ws)[:len(route)] == route
    _run(T, d, F, up)


@pytest.mark.parametrize("T,d,F,up", [(700, 192, 576, True), (1100, 128, 320, False), (1100, 128, 320, True)])
def test_weight_gradients_are_added_to(T, d, F, up):
    _run(T, d, F, up, accumulate=True)


def _backward(T, d, F, up, want_dx, grad=None, over=None):
    """The backward pass; with `grad` and `over`, that gradient starts where that buffer does."""
    s = inputs.StemShape("over", d, F, 300, 1, T, "bf16")
    bf, f32 = torch.bfloat16, torch.float32
    inp = inputs.layer_inputs(s, seed=73, device=DEV, tokens=T)
    put = {"W_gate": inp["W_gate"], "dy": inp["dy"], "H": inputs.normal((T, F), 0.5, 74, bf, DEV), "dV": (T, F),
           "dW_gate": (F, d), **({"W_up": inputs.normal((F, d), 0.02, 75, bf, DEV), "dW_up": (F, d)} if up else {})}
    shared = torch.empty(max(F * d * 4, T * F * 2), dtype=torch.uint8, device=DEV)
    b = {}
    for k, v in put.items():
        shape, dt = tuple(getattr(v, "shape", v)), f32 if k in ("dW_gate", "dW_up") else bf
        n = shape[0] * shape[1] * (4 if dt is f32 else 2)
        b[k] = shared[:n].view(dt).view(shape) if k in (grad, over) else torch.empty(shape, dtype=dt, device=DEV)
        if torch.is_tensor(v):
            b[k].copy_(v)
    G = inputs.normal((T, F), 1.0, 76, bf, DEV)
    dx = torch.empty(T, d, dtype=bf, device=DEV) if want_dx else None
    dWd = torch.empty(d, F, dtype=f32, device=DEV)
    ctx = Hn.make_ctx(s, T, reserve=L.STEM_RESERVE_UP if up else 0)
    a = (ctx, b["dy"], inp["x"], inp["ids"], b["W_gate"])
    if up:
        L.stem_ffn_up_backward(*a, b["W_up"], inp["W_down"], inp["E"], G, inputs.normal((T, F), 1.0, 77, bf, DEV), b["H"], dx,
                               b["dW_gate"], b["dW_up"], dWd, b["dV"])
    else:
        L.stem_ffn_backward(*a, inp["W_down"], inp["E"], G, b["H"], dx, b["dW_gate"], dWd, b["dV"])
    L.stem_sync_status(ctx)
    ctx.close()
    return {"dW_down": dWd, "dW_gate": b["dW_gate"], **({"dx": dx} if want_dx else {}), **({"dW_up": b["dW_up"]} if up else {})}


@pytest.mark.parametrize("up,grad,over,want_dx", [
    (False, "dW_gate", "H", True), (False, "dW_gate", "dy", True), (False, "dW_gate", "W_gate", True),
    (False, "dW_gate", "W_gate", False),
    (True, "dW_gate", "H", True), (True, "dW_gate", "dy", False), (True, "dW_gate", "W_gate", True), (True, "dW_gate", "W_up", True),
    (True, "dW_up", "H", False), (True, "dW_up", "dy", True), (True, "dW_up", "W_gate", True), (True, "dW_up", "W_up", True),
])
def test_gradient_over_a_buffer_that_was_read_before_it(up, grad, over, want_dx):
    """Layers whose gradients share a launch of several rounds of whole tiles (no K slices, whose sum would come after every
    read): there the first tiles of a gradient are stored long before the last ones of dW_down are read, and all of them
    before dx.  The gradients must be those of buffers that lie apart."""
    T, d, F = (473, 1920, 7232) if up else (1999, 2048, 8192)
    assert Hn.route_weight_grads(T, d, F, 3 if up else 2, min(64 << 20, 32 * d * max(T, F))) == (1, 256, 256, 1)
    assert (F // 256) * (d // 256) * (3 if up else 2) > 256
    want, got = _backward(T, d, F, up, want_dx), _backward(T, d, F, up, want_dx, grad, over)
    for k in want:   # the same tiles of the same length, in one launch or several
        assert torch.equal(want[k], got[k]), (k, float((want[k].float() - got[k].float()).abs().max()))
