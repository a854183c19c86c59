"""The few-row kernel's K slices: each workgroup of a tile finishes a share of its rows, or leaves it to the last to arrive."""
import ctypes

import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

DEV = "cuda:0"

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,F,slices", [
    (129, 1408, 2112, 4),     # a second token tile with one row: three of its shares are empty; 33 K tiles
    (256, 2048, 8192, 4),     # 256 workgroups
    (250, 1536, 5120, 4),
    (385, 1344, 2112, 2),     # a last token tile with one row, 33 K tiles in slices of 16 and 17
    (512, 1024, 2624, 4),
    (40, 4160, 2112, 2),      # one token tile, a third full
])
def test_shares_waited_for_and_left_behind(T, d, F, slices):
    assert Hn.route_forward(T, d, F)[1] == (Hn.FEW_ROW, 128, 64, slices)
    V = 300
    s = inputs.StemShape("slice-shares", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=81, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    a = (ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"])
    y, yr = torch.empty_like(inp["x"]), torch.empty_like(inp["x"])
    L.stem_ffn_forward(*a, y)
    L.stem_ffn_forward_residual(*a, inp["x"], yr)
    L.stem_sync_status(ctx)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    yo, _ = O.ffn_forward(f64["x"], inp["ids"].cpu().numpy(), f64["W_gate"], f64["W_down"], f64["E"])
    assert Hn.max_rel(y.float().cpu(), yo) <= Hn.TOL["bf16"]
    assert Hn.max_rel(yr.float().cpu(), f64["x"] + yo) <= Hn.TOL["bf16"]
    # The same bits whoever adds a share, and whatever the launches before: nobody waits, one look, some, as in use.
    for polls in (0, 1, 3, 0, 2000, 0, 2000):
        L.lib().stem_exchange_polls(ctx.handle, polls)
        for _ in range(4):
            out, xr = torch.empty_like(y), inp["x"].clone()
            L.stem_ffn_forward(*a, out)
            L.stem_ffn_forward_residual(ctx, xr, *a[2:], xr, xr)    # in place: a row added twice would show
            assert torch.equal(out, y) and torch.equal(xr, yr)
    ctx.close()


def test_slices_of_products_of_several_sizes_count_on_one_word():
    """Calls of few and many tokens on one context use the same words with two and with four slices."""
    d, F, V = 1408, 2112, 300
    s = inputs.StemShape("slice-words", d, F, V, 1, 512, "bf16")
    inp = inputs.layer_inputs(s, seed=82, device=DEV, tokens=512)
    ctx = Hn.make_ctx(s, 512)
    sizes = (129, 512, 200, 385, 256)
    assert {Hn.route_forward(T, d, F)[1][3] for T in sizes} == {2, 4}

    def forward(T):
        y = torch.empty(T, d, dtype=torch.bfloat16, device=DEV)
        L.stem_ffn_forward(ctx, inp["x"][:T], inp["ids"][:T], inp["W_gate"], inp["W_down"], inp["E"], y)
        return y

    first = {T: forward(T) for T in sizes}
    for T in sizes[::-1] + sizes:
        assert torch.equal(forward(T), first[T])
    graph, ys = torch.cuda.CUDAGraph(), {}
    with torch.cuda.graph(graph):
        for T in sizes:
            ys[T] = torch.empty(T, d, dtype=torch.bfloat16, device=DEV)
            L.stem_ffn_forward(ctx, inp["x"][:T], inp["ids"][:T], inp["W_gate"], inp["W_down"], inp["E"], ys[T],
                               stream=torch.cuda.current_stream())
    for _ in range(4):
        graph.replay()
        torch.cuda.synchronize()
        for T in sizes:
            assert torch.equal(ys[T], first[T])
            ys[T].zero_()
        forward(200)
    ctx.close()


@pytest.mark.parametrize("T,d,F,slices", [(129, 1408, 2112, 4), (256, 2048, 8192, 4), (385, 1344, 2112, 2)])
def test_output_over_what_the_slices_read(T, d, F, slices):
    """y inside the buffer that H is saved to, or over W_down: as if every slice had read all of it before y is written."""
    assert Hn.route_forward(T, d, F)[1] == (Hn.FEW_ROW, 128, 64, slices)
    s = inputs.StemShape("slice-over", d, F, 300, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=84, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    want, H = torch.empty_like(inp["x"]), torch.empty(T, F, dtype=torch.bfloat16, device=DEV)
    L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], want, None, H)
    n = T * d
    for at in (0, n // 16 * 8, T * F - n):                     # y in H: its beginning, its middle, its end
        room = torch.zeros(T * F, dtype=torch.bfloat16, device=DEV)
        y = room[at:at + n].view(T, d)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], y, None, room.view(T, F),
                               stream=torch.cuda.current_stream())
        for replay in (False, True, True):
            room.zero_()
            if replay:
                graph.replay()
            else:
                L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], y, None, room.view(T, F))
            torch.cuda.synchronize()
            assert torch.equal(y, want)
            left = torch.ones(T * F, dtype=torch.bool, device=DEV)
            left[at:at + n] = False
            assert torch.equal(room[left], H.view(-1)[left])   # what y does not cover of H
    for at in (0, F * d - 8):                                  # y over W_down's beginning, and over its last 16 bytes
        room = torch.zeros(F * d + n, dtype=torch.bfloat16, device=DEV)
        room[:F * d].copy_(inp["W_down"].view(-1))
        y = room[at:at + n].view(T, d)
        L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], room[:F * d].view(d, F), inp["E"], y)
        assert torch.equal(y, want)
    L.stem_sync_status(ctx)
    ctx.close()


@pytest.mark.parametrize("T,d,F", [
    (112, 1024, 3904),        # the fewest tokens, 7.99 MB of weights
    (128, 2048, 8192),        # all lines of the largest, four by each thread
    (129, 1536, 5184),        # just below the most from 129 tokens on
    (384, 1536, 5120),        # few-row gate product
    (128, 16000, 1024),       # the decode kernel's grid comes to 16.8 of 32.8 MB
    (300, 6144, 1216),        # the few-row kernel's to 11.2 of 14.9 MB
])
def test_gate_product_that_touches_the_down_products_weights(T, d, F):
    assert L.lib().stem_route_touch_bytes(d, F, ctypes.c_int64(T)) == 2 * d * F
    V = 300
    s = inputs.StemShape("touch", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=83, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    y, G, H = (torch.empty(T, n, dtype=torch.bfloat16, device=DEV) for n in (d, F, F))
    L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], y, G, H)
    L.stem_sync_status(ctx)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    yo, fw = O.ffn_forward(f64["x"], inp["ids"].cpu().numpy(), f64["W_gate"], f64["W_down"], f64["E"])
    for got, want in ((y, yo), (G, fw["g"]), (H, fw["h"])):
        assert Hn.max_rel(got.float().cpu(), want) <= Hn.TOL["bf16"]
    ctx.close()
