"""Gate and up product in one launch, and as two where the buffers ask for it."""
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

DEV = "cuda:0"

pytestmark = pytest.mark.gpu


def _layer(T, d, F, seed):
    s = inputs.StemShape("gate-up", d, F, 300, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=seed, device=DEV, tokens=T)
    inp["W_up"] = inputs.normal((F, d), 0.05, seed + 1, torch.bfloat16, DEV)
    return inp, Hn.make_ctx(s, T, reserve=L.STEM_RESERVE_UP)


def _forward(ctx, inp, E, G, Up, H, W_up=None):
    y = torch.empty_like(inp["x"])
    L.stem_ffn_up_forward(ctx, inp["x"], inp["ids"] if E is not None else None, inp["W_gate"],
                          inp["W_up"] if W_up is None else W_up, inp["W_down"], E, y, G, Up, H)
    L.stem_sync_status(ctx)
    return y


@pytest.mark.parametrize("T,d,F,tile", [
    (1, 64, 64, (128, 128)),           # one row, one K tile; the second wavefront's columns outside
    (130, 704, 2368, (128, 128)),      # a second row block with two rows
    (900, 1280, 3136, (192, 128)),     # 64 columns per tile; a last row block with 132 rows
    (1500, 576, 2112, (256, 128)),
    (1990, 1024, 4032, (256, 256)),    # 128 columns per tile, the last half outside; a row block with 198 rows
])
def test_gate_and_up_product_on_every_tiling(T, d, F, tile):
    assert Hn.route_tiles(T, 2 * F, d, 1, Hn.EPI_GATE)[1:3] == tile
    inp, ctx = _layer(T, d, F, 95)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    ids = inp["ids"].cpu().numpy()
    for E in (inp["E"], None):
        G, Up, H = (torch.full((T + 1, F), 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(3))
        y = _forward(ctx, inp, E, G[:T], Up[:T], H[:T])
        yo, fw = O.up_forward(f64["x"], ids, f64["W_gate"], f64["W_up"], f64["W_down"], f64["E"] if E is not None else None)
        ref = {"y": yo, "g": fw["g"], "h": fw["h"], "up": f64["x"] @ f64["W_up"].T}
        errs = {k: Hn.max_rel(v.float().cpu(), ref[k]) for k, v in (("y", y), ("g", G[:T]), ("h", H[:T]), ("up", Up[:T]))}
        assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
        assert all(bool((t[T] == 7.0).all()) for t in (G, Up, H))
        assert torch.equal(_forward(ctx, inp, E, None, None, None), y)       # nothing saved
    ctx.close()


def test_gate_and_up_product_over_each_other_and_over_what_they_read():
    T, d, F = 300, 256, 832
    inp, ctx = _layer(T, d, F, 96)
    E = inp["E"]
    G, Up, H = (torch.empty(T, F, dtype=torch.bfloat16, device=DEV) for _ in range(3))
    y = _forward(ctx, inp, E, G, Up, H)
    same = torch.empty_like(G)
    assert torch.equal(_forward(ctx, inp, E, same, same, None), y) and torch.equal(same, G)     # G stays where Up was
    assert torch.equal(_forward(ctx, inp, E, None, same, same), y) and torch.equal(same, H)     # H stays where Up was
    # W_up inside the buffer that G or H is stored to
    for at in range(2):
        room = torch.empty(T * F + F * d, dtype=torch.bfloat16, device=DEV)
        w = room[T * F // 2 // 8 * 8:][:F * d].view(F, d)
        w.copy_(inp["W_up"])
        out = room[:T * F].view(T, F)
        assert torch.equal(_forward(ctx, inp, E, out if at == 0 else None, Up, out if at else None, w), y)
        assert torch.equal(out, H if at else G)
    ctx.close()


@pytest.mark.parametrize("T,d,F,tile,split", [
    (390, 3072, 2112, (128, 128), True),      # the up product in two K slices, whose sum is stored when all have read W_up
    (1345, 576, 4096, (192, 128), False),
    (1500, 320, 4160, (256, 128), False),
    (1990, 320, 4160, (256, 256), False),
])
@pytest.mark.parametrize("table", [True, False])
def test_outputs_over_w_up_take_two_launches_on_every_tiling(T, d, F, tile, split, table):
    assert Hn.route_tiles(T, F, d, 1, Hn.EPI_GATE)[1:3] == tile
    assert (Hn.route_tiles(T, F, d, 1, Hn.EPI_BF16, L.lib().stem_route_splitk_bytes(d, F, T))[3] > 1) == split
    inp, ctx = _layer(T, d, F, 97)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    yo, fw = O.up_forward(f64["x"], inp["ids"].cpu().numpy(), f64["W_gate"], f64["W_up"], f64["W_down"], f64["E"] if table else None)
    ref = {"G": fw["g"], "Up": fw["up"], "H": fw["h"]}
    E = inp["E"] if table else None
    for over in [None, "G", "H"] + (["Up"] if split else []):
        out = {k: torch.empty(T, F, dtype=torch.bfloat16, device=DEV) for k in ref}
        w = inp["W_up"]
        if over:
            room = torch.empty(T * F + F * d, dtype=torch.bfloat16, device=DEV)
            w = room[T * F // 2 // 8 * 8:][:F * d].view(F, d)
            w.copy_(inp["W_up"])
            out[over] = room[:T * F].view(T, F)
        at = {k: v.data_ptr() for k, v in out.items()}
        if table:
            at.update(E=E.data_ptr(), ids=inp["ids"].data_ptr())
        assert Hn.route_gate_up_together(T, d, F, E.shape[0] if table else 0, W_up=w.data_ptr(), **at) == (over is None)
        y = _forward(ctx, inp, E, out["G"], out["Up"], out["H"], w)
        errs = {k: Hn.max_rel(out[k].float().cpu(), v) for k, v in ref.items()}
        errs["y"] = Hn.max_rel(y.float().cpu(), yo)
        assert all(v <= Hn.TOL["bf16"] for v in errs.values()), (over, errs)
    ctx.close()


@pytest.mark.parametrize("T,d,F,tile", [(130, 704, 2368, (128, 128)), (1990, 1024, 4032, (256, 256))])
def test_ids_outside_the_table_in_the_joint_launch(T, d, F, tile):
    assert Hn.route_tiles(T, 2 * F, d, 1, Hn.EPI_GATE)[1:3] == tile
    inp, ctx = _layer(T, d, F, 98)
    E_rows = inp["E"].shape[0]
    bad = inp["ids"].clone()
    bad[0], bad[T // 2], bad[-1] = -1, 2 ** 31 - 1, E_rows
    y = torch.empty_like(inp["x"])
    L.stem_ffn_up_forward(ctx, inp["x"], bad, inp["W_gate"], inp["W_up"], inp["W_down"], inp["E"], y)
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    inp["ids"] = bad.clamp(0, E_rows - 1)
    assert torch.equal(_forward(ctx, inp, inp["E"], None, None, None), y)
    ctx.close()
