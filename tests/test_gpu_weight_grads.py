"""Weight gradients that share a launch, against the oracle, on every tiling and K split; and where they may not share one."""
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(T, d, F, up, accumulate=False, alias=None):
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
        if alias == "H":
            dWg = H.view(torch.float32).flatten()[:F * d].view(F, d)
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


def test_gate_gradient_over_the_saved_activations():
    """dW_gate may lie over H, which dW_down has read by then: the products then follow each other."""
    _run(1100, 128, 320, False, alias="H")
