"""GPU parity at the edges of the tile shapes the bf16 products choose from."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# the joint gate and up product of the layers with an up projection
GATE_UP_TILE = {(1000, 512, 4160): (256, 256), (1300, 1152, 6016): (256, 128), (520, 64, 8192): (128, 128), (385, 128, 128): (128, 128),
                (600, 512, 2112): (128, 128), (1535, 1088, 4032): (256, 256), (1345, 576, 4096): (256, 256)}


# tile and K slices of dH (and the gate product beyond 512 tokens), dx, dx of two operand pairs, the weight gradients
@pytest.mark.parametrize("T,d,F,routes", [
    # ragged last tiles; the last of 8 slices of 9 K tiles has two
    (1000, 512, 4160, [(256, 128, 1), (128, 128, 8), (128, 128, 8), (128, 128, 1)]),
    # a ragged last K tile in the weight gradients
    (1300, 1152, 6016, [(256, 256, 1), (128, 128, 2), (256, 128, 4), (256, 128, 1)]),
    # one K tile, fewer than the stages in LDS
    (520, 64, 8192, [(256, 128, 1), (128, 128, 8), (128, 128, 8), (128, 128, 1)]),
    # two K tiles, one row in the last tile
    (385, 128, 128, [(128, 128, 1), (128, 128, 1), (128, 128, 1), (128, 128, 1)]),
    # 33 K tiles in 7 slices of 5, the last of 3; with two operand pairs 4 slices of 9 each
    (600, 512, 2112, [(128, 128, 1), (128, 128, 7), (128, 128, 8), (128, 128, 1)]),
])
@pytest.mark.parametrize("up", [False, True])
def test_bf16_products_on_every_tiling(T, d, F, routes, up, table=True):
    """Forward and backward of the layer, and (up) of the additive variant, whose dx product sums two operand
    pairs and cuts them into K slices; without `table`, of the dense layer."""
    assert [r[1:] for r in (Hn.route_tiles(T, F, d, 1, Hn.EPI_DH), Hn.route_tiles(T, d, F), Hn.route_tiles(T, d, F, 2),
                            Hn.route_tiles(F, d, T, 1, Hn.EPI_F32))] == routes
    if T > 512:
        assert Hn.route_forward(T, d, F) == ((Hn.TILES, *routes[0]), (Hn.TILES, *routes[1]))
    if up:
        assert Hn.route_tiles(T, 2 * F, d, 1, Hn.EPI_GATE)[1:3] == GATE_UP_TILE[T, d, F]
    V = 300
    s = inputs.StemShape("tilings", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=61, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T, reserve=L.STEM_RESERVE_UP if up else 0)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    ids = inp["ids"].cpu().numpy()
    if not up:
        out = Hn.hip_forward_backward(ctx, inp)
        y, _ = O.ffn_forward(f64["x"], ids, f64["W_gate"], f64["W_down"], f64["E"])
        bw = O.ffn_backward(f64["dy"], f64["x"], ids, f64["W_gate"], f64["W_down"], f64["E"])
        ref = {"y": y, "dx": bw["dx"], "dU": bw["dU"], "dW_gate": bw["dW_gate"], "dW_down": bw["dW_down"]}
    else:
        Wu = inputs.normal((F, d), 0.02, 62, torch.bfloat16, DEV)
        e = lambda *sh, dt=torch.bfloat16: torch.empty(*sh, dtype=dt, device=DEV)  # noqa: E731
        out = {"y": e(T, d), "dx": e(T, d), "dU": e(T, F), "dW_gate": e(F, d, dt=torch.float32),
               "dW_up": e(F, d, dt=torch.float32), "dW_down": e(d, F, dt=torch.float32)}
        G, Up, H = e(T, F), e(T, F), e(T, F)
        E, e64 = (inp["E"], f64["E"]) if table else (None, None)
        L.stem_ffn_up_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], Wu, inp["W_down"], E, out["y"], G, Up, H)
        L.stem_ffn_up_backward(ctx, inp["dy"], inp["x"], inp["ids"], inp["W_gate"], Wu, inp["W_down"], E, G, Up, H,
                               out["dx"], out["dW_gate"], out["dW_up"], out["dW_down"], out["dU"])
        wu = inputs.to_f64(Wu)
        y, fw = O.up_forward(f64["x"], ids, f64["W_gate"], wu, f64["W_down"], e64)
        bw = O.up_backward(f64["dy"], f64["x"], ids, f64["W_gate"], wu, f64["W_down"], e64)
        out.update(G=G, Up=Up, H=H)
        ref = {"G": fw["g"], "Up": fw["up"], "H": fw["h"], "y": y, "dx": bw["dx"], "dU": bw["dV"], "dW_gate": bw["dW_gate"], "dW_up": bw["dW_up"], "dW_down": bw["dW_down"]}
    L.stem_sync_status(ctx)
    errs = {k: Hn.max_rel(out[k].float().cpu(), v) for k, v in ref.items()}
    assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
    ctx.close()


@pytest.mark.parametrize("T,d,F,routes,up", [
    (1345, 576, 4096, [(192, 128, 1), (128, 128, 4), (128, 128, 4), (128, 128, 1)], False),   # one row in the last tile; 9 K tiles
    (1535, 1088, 4032, [(192, 128, 1), (128, 128, 2), (128, 128, 2), (256, 128, 1)], True),   # ragged in both, a dense third row block
    (1345, 1024, 8128, [(256, 256, 1), (192, 128, 4), (256, 128, 4), (256, 128, 1)], False),  # slices of 32 K tiles, the last of 31
    (2690, 1984, 640, [(128, 128, 1), (192, 128, 1), (256, 128, 1), (128, 128, 2)], False),   # plain products, unsplit
])
def test_bf16_products_on_192_row_tiles(T, d, F, routes, up):
    test_bf16_products_on_every_tiling(T, d, F, routes, up)


@pytest.mark.parametrize("T,d,F,routes", [
    (1535, 1088, 4032, [(192, 128, 1), (128, 128, 2), (128, 128, 2), (256, 128, 1)]),
    (1345, 576, 4096, [(192, 128, 1), (128, 128, 4), (128, 128, 4), (128, 128, 1)]),
])
def test_dense_layers_on_192_row_tiles(T, d, F, routes):
    test_bf16_products_on_every_tiling(T, d, F, routes, up=True, table=False)


def test_residual_on_192_row_tiles():
    T, d, F = 2690, 1984, 640
    inp = inputs.layer_inputs(inputs.StemShape("res", d, F, 300, 1, T, "bf16"), seed=67, device=DEV, tokens=T)
    ctx = Hn.make_ctx(inputs.StemShape("res", d, F, 300, 1, T, "bf16"), T)
    a = (ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"])
    y, yr = torch.empty_like(inp["x"]), torch.empty_like(inp["x"])
    L.stem_ffn_forward(*a, y)
    L.stem_ffn_forward_residual(*a, inp["x"], yr)
    L.stem_sync_status(ctx)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    yo, _ = O.ffn_forward(f64["x"], inp["ids"].cpu().numpy(), f64["W_gate"], f64["W_down"], f64["E"])
    assert Hn.max_rel(y.float().cpu(), yo) <= Hn.TOL["bf16"]
    assert Hn.max_rel(yr.float().cpu(), f64["x"] + yo) <= Hn.TOL["bf16"]
    ctx.close()


@pytest.mark.parametrize("T,d,F", [
    (1030, 1028, 1028),   # every product on 32x32 tiles with one K tile in flight, ragged in M, N and K
    (1030, 36, 1028),     # forward and dH with K of one tile and a bit; dx, weight gradients with two K tiles in flight
    (33, 4, 8),           # K of one 16-byte piece, one row in the last tile
    (2030, 1004, 2044),   # every product on 64x64 tiles, ragged in M, N and K
    (1000, 256, 1028),    # the products behind dG in one launch of more than 512 workgroups
    (2030, 36, 1020),     # forward and dH on 64x64 tiles with fewer K tiles than wavefronts
])
def test_f32_products_on_both_tilings(T, d, F):
    s = inputs.StemShape("f32-tilings", d, F, 300, 1, T, "f32")
    inp = inputs.layer_inputs(s, seed=63, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    ids = inp["ids"].cpu().numpy()
    out = Hn.hip_forward_backward(ctx, inp)
    y2 = torch.empty_like(out["y"])
    L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], y2)   # G and H not saved
    acc = {k: out[k].clone() for k in ("dW_gate", "dW_down")}
    dU2, dx2 = torch.empty_like(out["dU"]), torch.empty_like(out["dx"])
    L.stem_ffn_backward(ctx, inp["dy"], inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], out["G"], None, dx2,
                        acc["dW_gate"], acc["dW_down"], dU2, accumulate=True)
    L.stem_sync_status(ctx)
    y, fw = O.ffn_forward(f64["x"], ids, f64["W_gate"], f64["W_down"], f64["E"])
    bw = O.ffn_backward(f64["dy"], f64["x"], ids, f64["W_gate"], f64["W_down"], f64["E"])
    ref = {"y": y, "G": fw["g"], "H": fw["h"], "dx": bw["dx"], "dU": bw["dU"], "dW_gate": bw["dW_gate"], "dW_down": bw["dW_down"]}
    errs = {k: Hn.max_rel(out[k].cpu(), v) for k, v in ref.items()}
    errs.update({k + " added": Hn.max_rel(v.cpu(), 2 * ref[k]) for k, v in acc.items()})
    assert all(v <= Hn.TOL["f32"] for v in errs.values()), errs
    assert torch.equal(out["y"], y2) and torch.equal(out["dU"], dU2) and torch.equal(out["dx"], dx2)
    ctx.close()


# tile and K slices of the gate and the down product
@pytest.mark.parametrize("T,d,F,gate,down", [
    (1, 64, 64, (16, 16, 1), (16, 16, 1)),          # one K tile: fewer than wavefronts and than K tiles in flight
    (16, 192, 4160, (16, 32, 1), (16, 16, 2)),      # 65 K tiles in slices of 33 and 32
    (17, 128, 8192, (32, 32, 1), (32, 16, 8)),      # one token in the second fragment
    (33, 64, 4096, (64, 16, 1), (64, 16, 4)),
    (129, 1088, 2112, (64, 32, 1), (64, 16, 1)),    # three token tiles, the last with one row
    (64, 2048, 8256, (64, 64, 1), (64, 16, 2)),     # 129 K tiles in slices of 65 and 64; a ragged last weight tile
    (20, 1024, 4160, (32, 32, 1), (32, 16, 4)),     # 65 K tiles in four slices, the last of 14
    (500, 512, 1536, (64, 64, 1), (64, 16, 1)),     # eight token tiles, the last ragged
    (300, 1024, 2624, (64, 64, 1), "few"),          # the down product on the few-row kernel beyond 256 tokens
    (250, 2048, 8192, "few", "few"),                # both there, a ragged second token tile
])
def test_decode_products_on_every_tile(T, d, F, gate, down):
    for got, want in zip(Hn.route_forward(T, d, F), (gate, down)):
        assert got[0] == Hn.FEW_ROW if want == "few" else got == (Hn.DECODE, *want)
    V = 300
    s = inputs.StemShape("decode-tiles", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=65, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    L.lib().stem_exchange_two_launches(ctx.handle, 1)   # (up to 32 tokens: what serves calls that are not one launch)
    a = (ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"])
    e = lambda n: torch.empty(T, n, dtype=torch.bfloat16, device=DEV)  # noqa: E731
    y, G, H, yr, xr = e(d), e(F), e(F), e(d), inp["x"].clone()
    assert Hn.kernels(ctx, lambda: L.stem_ffn_forward(*a, y, G, H)) == {"gemm_gate_fused": 1, "gemm_down": 1}
    L.stem_ffn_forward_residual(*a, inp["x"], yr)
    L.stem_ffn_forward_residual(ctx, xr, *a[2:], xr, xr)                # in place
    reps = [torch.empty_like(y) for _ in range(3)]
    for r in reps:
        L.stem_ffn_forward(*a, r)
    L.stem_sync_status(ctx)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    yo, fw = O.ffn_forward(f64["x"], inp["ids"].cpu().numpy(), f64["W_gate"], f64["W_down"], f64["E"])
    ref = {"y": yo, "G": fw["g"], "H": fw["h"], "yr": f64["x"] + yo}
    errs = {k: Hn.max_rel(v.float().cpu(), ref[k]) for k, v in (("y", y), ("G", G), ("H", H), ("yr", yr))}
    assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
    assert torch.equal(yr, xr) and all(torch.equal(r, y) for r in reps)
    ctx.close()


@pytest.mark.parametrize("T,d,F,gate,down", [
    (1, 64, 832, (16, 16, 1), (8, 8, 1)),           # 6.5 K tiles of 128, the fewest, for 8 wavefronts; eight weight tiles
    (1, 64, 768, (16, 16, 1), (16, 16, 1)),         # fewer, which whole fragments multiply faster
    (1, 64, 128, (16, 16, 1), (16, 16, 1)),
    (8, 2048, 8192, (16, 32, 1), (8, 8, 1)),        # the most tokens, weight tiles and K tiles in flight
    (7, 1088, 2176, (16, 16, 1), (8, 8, 1)),        # 17 K tiles over 8 wavefronts
    (3, 192, 4224, (16, 32, 1), (8, 8, 1)),         # 33: one wavefront has a fifth
    (8, 512, 1344, (16, 16, 1), (8, 8, 1)),         # 10.5 K tiles of 128
    (2, 64, 960, (16, 16, 1), (8, 8, 1)),           # 7.5
    (2, 64, 192, (16, 16, 1), (16, 16, 1)),
    (5, 2112, 1024, (16, 16, 1), (16, 16, 1)),      # more weight rows than 256 workgroups of 8
    (9, 256, 1024, (16, 16, 1), (16, 16, 1)),       # a ninth token
])
def test_down_product_of_up_to_eight_tokens(T, d, F, gate, down):
    test_decode_products_on_every_tile(T, d, F, gate, down)


SORT_KERNELS = [{"sort_fused"}, {"sort_fused"}, {"sort_fused", "sort_merge", "unique"}, {"sort_fused", "sort_merge", "unique"},
                {"sort_count", "sort_scan", "sort_scatter", "unique"}]


def _sort(ctx, ids, route, dU=None):
    """The names of the kernels of a table gradient whose sorted ids take the ids' place (not in the digit passes, which may read them
    meanwhile), and its outputs."""
    dev = torch.from_numpy(ids).to(DEV)
    e = lambda n: torch.empty(n, dtype=torch.int32, device=DEV)  # noqa: E731
    T, cap = len(ids), min(len(ids), ctx.vocab)
    out = dict(sorted_ids=dev if route != Hn.SORT_DIGITS else e(T), perm=e(T), uniq_ids=e(cap), seg_offsets=e(cap + 1), n_uniq=e(1))
    lie = {k: v.data_ptr() for k, v in out.items()}
    assert not Hn.route_sort_ranks(T, ctx.vocab, ids=dev.data_ptr(), **lie) and not Hn.route_sort_buckets(T, ctx.vocab, ids=dev.data_ptr(), **lie)
    out["dE_rows"] = None if dU is None else torch.empty(cap, ctx.d_ff, dtype=torch.float32, device=DEV)
    seen = Hn.kernels(ctx, lambda: L.stem_embed_grad(ctx, dev, dU, *out.values()))
    return {k for k in seen if not k.startswith("seg")}, out


@pytest.mark.parametrize("T,V,route", [
    (1, 1, Hn.SORT_ONE_1024), (63, 2, Hn.SORT_ONE_1024), (1024, 128256, Hn.SORT_ONE_1024), (1025, 128256, Hn.SORT_ONE_4096),
    (4096, 1 << 20, Hn.SORT_ONE_4096), (4097, 1 << 20, Hn.SORT_RUNS_1024),
    (4096, (1 << 20) + 1, Hn.SORT_RUNS_1024),            # an id that leaves no room for 12 position bits
    (16384, (1 << 18) + 1, Hn.SORT_RUNS_1024), (16384, 50304, Hn.SORT_RUNS_1024), (16385, 50304, Hn.SORT_RUNS_4096),   # the most runs of 1024; a last run with one key
    (65537, 128256, Hn.SORT_RUNS_4096), (262144, 7, Hn.SORT_RUNS_4096),   # more runs than searches in flight; long runs of equal ids
    (5000, 5_000_000, Hn.SORT_DIGITS), (262145, 3, Hn.SORT_DIGITS),       # ids, then a batch, beyond the merge's
])
def test_sort_on_every_path(T, V, route):
    """(Ranks and buckets of up to 16384 ids aside: the sorted ids go over the ids, which they leave to these kernels.)"""
    assert Hn.route_sort(T, V) == route
    ids = inputs.zipf_ids(T, V, seed=67)
    ids[T // 2:] = np.random.default_rng(68).integers(0, V, T - T // 2)
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    for turn in range(2):                                # the second call finds the first one's scratch
        seen, eg = _sort(ctx, ids, route)
        L.stem_sync_status(ctx)
        assert seen == SORT_KERNELS[route]
        Hn.check_integers(eg, ids)
        ids = ids[::-1].copy()
    ctx.close()


def test_f32_backward_without_dx_and_with_dx_over_its_inputs():
    """dx may take the place of dy, which the products before it have read: then they are launches of their own."""
    T, d, F = 300, 64, 192
    s = inputs.StemShape("f32-alias", d, F, 300, 1, T, "f32")
    inp = inputs.layer_inputs(s, seed=69, device=DEV, tokens=T)
    ctx = Hn.make_ctx(s, T)
    out = Hn.hip_forward_backward(ctx, inp)
    for dx in (None, inp["dy"]):
        g = {k: torch.empty_like(out[k]) for k in ("dW_gate", "dW_down", "dU")}
        L.stem_ffn_backward(ctx, inp["dy"], inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], out["G"], out["H"],
                            dx, g["dW_gate"], g["dW_down"], g["dU"])
        L.stem_sync_status(ctx)
        assert all(torch.allclose(g[k], out[k], rtol=0, atol=1e-6 * float(out[k].abs().max())) for k in g)
    assert torch.allclose(inp["dy"], out["dx"], rtol=0, atol=1e-6 * float(out["dx"].abs().max()))
    ctx.close()


def _sum_over_tokens(a, b):
    """a^T b, the wider operand in pieces of fewer than 2^31 elements (the library product behind torch needs that)."""
    if a.shape[1] > b.shape[1]:
        return _sum_over_tokens(b, a).T
    return torch.cat([a.T @ p.contiguous() for p in b.split(1 << 24, dim=1)], dim=1)


def _reference64(inp):
    """Forward and backward of the layer in 64-bit torch on the GPU (plain products; for layers too wide for the oracle's
    host arrays)."""
    x, dy, Wg, Wd, E = (inp[k].double() for k in ("x", "dy", "W_gate", "W_down", "E"))
    Er = E[inp["ids"].long()]
    G = x @ Wg.T
    s = torch.sigmoid(G)
    H, dH = G * s * Er, dy @ Wd
    dG = dH * Er * s * (1 + G * (1 - s))
    return {"y": H @ Wd.T, "G": G, "H": H, "dU": dH * G * s, "dx": dG @ Wg, "dW_gate": _sum_over_tokens(dG, x),
            "dW_down": _sum_over_tokens(dy, H)}


def _max_rel(got, ref):
    return float((got.double() - ref).abs().max() / ref.abs().max())


@pytest.mark.parametrize("T", [1, 65])   # a K tile of the weight gradients with 1 row, a second one with 1 row
@pytest.mark.parametrize("wide_d", [False, True])
def test_bf16_layer_with_the_longest_rows(T, wide_d):
    """64 x 8388544, just below 2^31 bytes of fp32 weight gradient: a K tile of [T, d_ff] is 1 GiB, so the three K
    tiles that the weight gradients' loaders request beyond the last one lie more than 2^31 bytes behind the operand."""
    d, F = (8388544, 64) if wide_d else (64, 8388544)
    s = inputs.StemShape("longest-rows", d, F, 3, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=71, device=DEV, tokens=T)
    if wide_d:   # gate activations of order one
        inp["W_gate"] *= 0.03
    ctx = Hn.make_ctx(s, T)
    out = Hn.hip_forward_backward(ctx, inp)
    L.stem_sync_status(ctx)
    errs = {k: _max_rel(out[k], v) for k, v in _reference64(inp).items()}
    assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
    ctx.close()


@pytest.mark.parametrize("T,d,F", [(3, 1 << 26, 8), (35, 8, (1 << 26) + 4)])
def test_f32_layer_with_rows_beyond_a_buffer_window(T, d, F):
    """Eight rows of 2^26 floats are 2 GiB.  Small integers times a power of two make the sums over d_model exact, a table
    of few nonzero columns those over d_ff short, so the tolerance is that of the other fp32 layers."""
    g = torch.Generator(device=DEV).manual_seed(73)
    r = lambda *sh: torch.randint(-1, 2, sh, generator=g, device=DEV, dtype=torch.int8).float()  # noqa: E731
    inp = {"x": r(T, d), "dy": r(T, d), "W_gate": r(F, d).mul_(2.0 ** -12 if d > F else 1.0),
           "W_down": r(d, F).mul_(2.0 ** -12 if d > F else 1.0), "E": torch.zeros(3, F, device=DEV),
           "ids": torch.arange(T, device=DEV, dtype=torch.int32) % 3}
    cols = torch.arange(F, device=DEV) if F < 100 else torch.cat([torch.tensor([0, 1, F - 2, F - 1], device=DEV),
                                                                   torch.randint(0, F, (500,), generator=g, device=DEV)])
    inp["E"][:, cols] = torch.randn(3, len(cols), generator=g, device=DEV)
    ctx = Hn.make_ctx(inputs.StemShape("f32-wide", d, F, 3, 1, T, "f32"), T)
    out = Hn.hip_forward_backward(ctx, inp)
    L.stem_sync_status(ctx)
    errs = {k: _max_rel(out[k], v) for k, v in _reference64(inp).items()}
    assert all(v <= Hn.TOL["f32"] for v in errs.values()), errs
    ctx.close()


BAD_IDS = [300, -3, 2 ** 31 - 1, -2 ** 31, 307, -1, 257, 300]


def _with_bad_ids(ids, at, V):
    bad = ids.copy()
    bad[at] = [b if b < 0 else max(b, V) for b in BAD_IDS]
    return bad, np.clip(bad.astype(np.int64), 0, V - 1)


def _expect_id_range(ctx):
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    L.stem_sync_status(ctx)   # the flag was cleared


@pytest.mark.parametrize("T,d,F,gate,wait", [
    # d_ff 64 modulo 128: the last column block of a wavefront is half outside; 9 K tiles: early touch of the table rows
    (1300, 576, 6208, (Hn.TILES, 256, 256), False),
    (900, 576, 4160, (Hn.TILES, 256, 128), False),
    (520, 576, 320, (Hn.TILES, 128, 128), False),
    # gather in the gate product's epilogue, and (wait) the plain product with the gather behind it
    (250, 1536, 5120, (Hn.FEW_ROW, 128, 64), False),
    (250, 1536, 5120, (Hn.FEW_ROW, 128, 64), True),
    (300, 128, 320, (Hn.DECODE, 64, 16), False),
    (300, 128, 320, (Hn.DECODE, 64, 16), True),
])
def test_out_of_range_ids_on_every_forward_kernel(T, d, F, gate, wait):
    """Ids outside the table read row 0 or the last one, are reported once, and leave everything else as it is: the
    results are those of the clamped ids."""
    V = 257
    assert Hn.route_forward(T, d, F)[0][:3] == gate
    s = inputs.StemShape("bad-ids", d, F, V, 1, T, "bf16")
    inp = inputs.layer_inputs(s, seed=75, device=DEV, tokens=T)
    ids, clamped = _with_bad_ids(inp["ids"].cpu().numpy(), [0, 5, 63, 64, 128, 249, T // 2, T - 1], V)
    inp["ids"] = torch.from_numpy(ids).to(DEV)
    f64 = {k: inputs.to_f64(v) for k, v in inp.items() if k != "ids"}
    y, fw = O.ffn_forward(f64["x"], clamped, f64["W_gate"], f64["W_down"], f64["E"])
    ref = {"y": y, "G": fw["g"], "H": fw["h"]}
    ctx = Hn.make_ctx(s, T)
    if gate[0] == Hn.TILES:
        assert Hn.route_tiles(T, F, d, 1, Hn.EPI_DH)[1:3] == gate[1:]
        # the forward call's report is collected first: the backward call would make it and do nothing else
        out = Hn.hip_forward_backward(ctx, inp, after_forward=lambda: _expect_id_range(ctx))
        bw = O.ffn_backward(f64["dy"], f64["x"], clamped, f64["W_gate"], f64["W_down"], f64["E"])
        ref.update({k: bw[k] for k in ("dx", "dU", "dW_gate", "dW_down")})
    else:
        out = {k: torch.empty(T, n, dtype=torch.bfloat16, device=DEV) for k, n in (("y", d), ("G", F), ("H", F))}
        ready = torch.cuda.Event()
        ready.record()
        L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], out["y"], out["G"], out["H"],
                           wait_event=ready.cuda_event if wait else None)
    _expect_id_range(ctx)
    errs = {k: Hn.max_rel(out[k].float().cpu(), v) for k, v in ref.items()}
    assert all(v <= Hn.TOL["bf16"] for v in errs.values()), errs
    ctx.close()


@pytest.mark.parametrize("T,V,route", [(1000, 300, Hn.SORT_ONE_1024), (4000, 300, Hn.SORT_ONE_4096), (16000, 300, Hn.SORT_RUNS_1024),
                                       (20000, 300, Hn.SORT_RUNS_4096), (5000, 5_000_000, Hn.SORT_DIGITS)])
def test_out_of_range_ids_on_every_sort(T, V, route):
    assert Hn.route_sort(T, V) == route
    ids, clamped = _with_bad_ids(inputs.zipf_ids(T, V, seed=76), [0, 7, 63, 64, 255, 256, T // 2, T - 1], V)
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    dU = inputs.normal((T, 64), 1.0, 77, torch.bfloat16, DEV)
    seen, eg = _sort(ctx, ids, route, dU)
    _expect_id_range(ctx)
    assert seen == SORT_KERNELS[route]
    clamped = clamped.astype(np.int32)
    U = Hn.check_integers(eg, clamped)
    assert Hn.max_rel(eg["dE_rows"][:U].cpu(), O.embed_grad(clamped, inputs.to_f64(dU))["dE_rows"]) <= 1e-5
    ctx.close()
