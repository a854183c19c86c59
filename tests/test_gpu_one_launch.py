"""A decode step's layer in one launch: at the edges of its tiles, in calls that follow each other with other sizes, where the workgroups
do not wait for each other, and replayed from a graph."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _layer(T, d, F, V, seed):
    n = lambda shape, std, k: inputs.normal(shape, std, seed + k, torch.bfloat16, DEV)
    ids = torch.from_numpy(inputs.zipf_ids(T, V, seed=seed)).to(DEV)
    return dict(x=n((T, d), 1.0, 1), ids=ids, Wg=n((F, d), 0.05, 2), Wd=n((d, F), 0.05, 3), E=n((V, F), 0.5, 4), r=n((T, d), 1.0, 5))


def _call(ctx, s, y, residual=True):
    if residual:
        L.stem_ffn_forward_residual(ctx, s["x"], s["ids"], s["Wg"], s["Wd"], s["E"], s["r"], y)
    else:
        L.stem_ffn_forward(ctx, s["x"], s["ids"], s["Wg"], s["Wd"], s["E"], y)
    return y


def _bound(s, ref):
    """What roundings to bf16 may do: H once (each product of the sum by 2^-9 of itself), y once; the fp32 sums' are far below."""
    f = {k: inputs.to_f64(s[k]) for k in ("x", "Wg", "Wd", "E")}
    h = O.ffn_forward(f["x"], s["ids"].cpu().numpy(), f["Wg"], np.eye(f["Wg"].shape[0]), f["E"])[0]
    return 2.0 ** -9 * (np.abs(h) @ np.abs(f["Wd"]).T) + 2.0 ** -8 * np.abs(ref) + 1e-4


SIZES = [(1, 64, 64), (8, 512, 2048), (9, 512, 2112), (16, 576, 64), (17, 1024, 4096), (32, 1024, 4160), (24, 1088, 2048), (7, 1536, 4096),
         (16, 1600, 8192), (1, 2048, 8192), (8, 2048, 2048), (9, 2048, 8192), (16, 2048, 8192), (24, 1536, 8192), (5, 64, 8192), (20, 64, 8128),
         (12, 2048, 64), (3, 1024, 1984), (32, 640, 2496), (31, 1024, 8192), (32, 512, 8192), (32, 512, 2048),
         # 24 columns of H a workgroup, the last one with 8 or 16 of them
         (6, 1280, 5120), (22, 1536, 5056), (15, 2048, 6144), (4, 192, 4160), (32, 1024, 6144)]


@pytest.mark.parametrize("T,d,F", SIZES)
def test_layer_in_one_launch_matches_the_oracle(T, d, F):
    assert L.lib().stem_route_one_launch(d, F, ctypes.c_int64(T))
    V = 300
    s = _layer(T, d, F, V, 100 + T)
    ctx = L.stem_create(d, F, V, L.STEM_BF16, T, 0)
    f = {k: inputs.to_f64(v) for k, v in s.items() if k != "ids"}
    ref, _ = O.ffn_forward(f["x"], s["ids"].cpu().numpy(), f["Wg"], f["Wd"], f["E"])
    new = lambda: torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    plain = new()
    assert Hn.kernels(ctx, lambda: _call(ctx, s, plain, residual=False)) == {"ffn_decode": 1}
    added = _call(ctx, s, new())
    L.stem_sync_status(ctx)
    for y, want in ((plain, ref), (added, ref + f["r"])):
        assert (np.abs(inputs.to_f64(y) - want) <= _bound(s, want)).all(), float((np.abs(inputs.to_f64(y) - want) / _bound(s, want)).max())
    # activations saved beside it
    G, H = (torch.full((T, F), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    kept = new()
    L.stem_ffn_forward(ctx, s["x"], s["ids"], s["Wg"], s["Wd"], s["E"], kept, G, H)
    g, e = f["x"] @ f["Wg"].T, f["E"][s["ids"].cpu().numpy()]
    assert torch.equal(kept, plain) and Hn.max_rel(G.float().cpu(), g) < 5e-3 and Hn.max_rel(H.float().cpu(), g / (1 + np.exp(-g)) * e) < 5e-3
    # in place on x, and again to the same bits
    again = dict(s, r=s["x"].clone())
    other = _call(ctx, again, new())
    inplace = s["x"].clone()
    _call(ctx, dict(s, x=inplace, r=inplace), inplace)
    assert torch.equal(other, inplace) and torch.equal(_call(ctx, s, new()), added)
    # nobody waits: all but the last workgroup give their rows up, and others do them; one look and some, after which they may take them
    # back; and as in use.  In place a row done twice would show, as the layer is added to it again.
    for looks in (0, 1, 3, 0, 12, 200):
        L.lib().stem_exchange_polls(ctx.handle, looks)
        for _ in range(3):
            assert torch.equal(_call(ctx, s, new()), added), looks
            inplace = s["x"].clone()
            _call(ctx, dict(s, x=inplace, r=inplace), inplace)
            assert torch.equal(other, inplace), looks
    L.stem_sync_status(ctx)
    ctx.close()


def test_calls_of_other_sizes_between_and_graph_replays():
    """One context, calls of 1 to 32 tokens with two launches (33 tokens) and calls that wait for an event (two launches too) between; replays."""
    d, F, V = 640, 2496, 300
    ctx = L.stem_create(d, F, V, L.STEM_BF16, 40, 0)
    cases = [_layer(T, d, F, V, 7 * T) for T in (32, 1, 33, 8, 24, 16, 9)]
    ys = [torch.zeros_like(c["x"]) for c in cases]
    want = []
    for c, y in zip(cases, ys):
        want.append(_call(ctx, c, y).clone())
        event, two = torch.cuda.Event(), torch.empty_like(y)
        event.record()
        L.stem_ffn_forward(ctx, c["x"], c["ids"], c["Wg"], c["Wd"], c["E"], two, wait_event=event.cuda_event)
        assert Hn.max_rel(_call(ctx, c, torch.empty_like(y), residual=False).float().cpu(), two.float().cpu()) < 2e-2
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for c, y in zip(cases, ys):
            _call(ctx, c, y)
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for c, y in zip(cases, ys):
            _call(ctx, c, y)
    for n in range(4):
        for y in ys:
            y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(ys, want)), n
        assert torch.equal(_call(ctx, cases[n], torch.empty_like(ys[n])), want[n])     # eager work between the replays
    L.stem_sync_status(ctx)
    ctx.close()


@pytest.mark.parametrize("T,d,F", [(3, 512, 1536), (16, 2048, 8192)])
def test_launch_numbers_wrap(T, d, F):
    """The calls about the 2^32-th of a context, eager and from a graph, waited for and given up."""
    assert L.lib().stem_route_one_launch(d, F, ctypes.c_int64(T))
    s = _layer(T, d, F, 300, 40)
    ctx = L.stem_create(d, F, 300, L.STEM_BF16, T, 0)
    want = s["x"].clone()
    _call(ctx, dict(s, x=want, r=want), want)
    x = s["x"].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _call(ctx, dict(s, x=x, r=x), x)
    for polls, replay in ((200, False), (200, True), (0, False)):
        L.lib().stem_exchange_polls(ctx.handle, polls)
        assert L.lib().stem_exchange_launch(ctx.handle, ctypes.c_uint32(2 ** 32 - 3)) == 0
        for n in range(5):
            x.copy_(s["x"])
            if replay:
                graph.replay()
            else:
                _call(ctx, dict(s, x=x, r=x), x)
            assert torch.equal(x, want), (polls, replay, n)
    L.stem_sync_status(ctx)
    ctx.close()


def test_two_contexts_on_two_streams_at_once():
    d, F, V, T = 1024, 4096, 500, 24
    ss = [_layer(T, d, F, V, 50 + i) for i in range(2)]
    ctxs = [L.stem_create(d, F, V, L.STEM_BF16, T, 0) for _ in ss]
    want = [_call(c, s, torch.empty_like(s["x"])) for c, s in zip(ctxs, ss)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ss]
    outs = [[torch.empty_like(s["x"]) for _ in range(40)] for s in ss]
    for n in range(40):
        for c, s, st, o in zip(ctxs, ss, streams, outs):
            with torch.cuda.stream(st):
                _call(c, s, o[n])
    torch.cuda.synchronize()
    for w, o in zip(want, outs):
        assert all(torch.equal(w, y) for y in o)
    for c in ctxs:
        L.stem_sync_status(c)
        c.close()


@pytest.mark.parametrize("T,d,F", [(1, 2048, 8192), (16, 2048, 8192), (32, 1024, 4096)])
def test_steps_on_four_streams_keep_each_other_going(T, d, F):
    """Workgroups wait for those of their launch, which other launches keep from the chip if no two fit a compute unit: a round of four steps
    then took fifty times as long as a step alone.  In turn it is four times."""
    layers, rounds = 4, 20
    s = _layer(T, d, F, 300, 60)
    ctxs, streams, graphs, xs = [], [], [], []
    want = None
    for _ in range(4):
        ctx, x = L.stem_create(d, F, 300, L.STEM_BF16, T, 0), s["x"].clone()
        step = lambda: [_call(ctx, dict(s, x=x, r=x), x) for _ in range(layers)]  # noqa: B023, E731
        step()
        torch.cuda.synchronize()
        want = x.clone() if want is None else want
        assert torch.equal(x, want)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            x.copy_(s["x"])
            step()
        ctxs.append(ctx), streams.append(torch.cuda.Stream()), graphs.append(g), xs.append(x)

    def us_a_round(n):
        torch.cuda.synchronize()
        ends = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
        start = torch.cuda.Event(enable_timing=True)
        start.record()
        for st in streams[:n]:
            st.wait_event(start)
        for _ in range(rounds):
            for g, st in zip(graphs[:n], streams):
                with torch.cuda.stream(st):
                    g.replay()
        for e, st in zip(ends, streams):
            e.record(st)
        torch.cuda.synchronize()
        return max(start.elapsed_time(e) for e in ends) * 1e3 / rounds

    us_a_round(4)
    one, four = sorted(us_a_round(1) for _ in range(3))[1], sorted(us_a_round(4) for _ in range(3))[1]
    assert four < 12 * one, (one, four)
    assert all(torch.equal(x, want) for x in xs)
    for c in ctxs:
        L.stem_sync_status(c)
    del graphs
    for c in ctxs:
        c.close()


def test_ids_outside_the_table_are_clamped_and_reported():
    d, F, V, T = 512, 2048, 100, 12
    s = _layer(T, d, F, V, 3)
    ctx = L.stem_create(d, F, V, L.STEM_BF16, T, 0)
    bad = s["ids"].clone()
    bad[0], bad[5], bad[11] = -1, V, 2 ** 31 - 1
    y = _call(ctx, dict(s, ids=bad), torch.empty_like(s["x"]))
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    assert torch.equal(y, _call(ctx, dict(s, ids=bad.clamp(0, V - 1)), torch.empty_like(y)))
    L.stem_sync_status(ctx)
    ctx.close()


@pytest.mark.parametrize("T,d,F", [(5, 64, 8256), (16, 64, 8256), (20, 64, 8256), (9, 2112, 1024), (20, 2112, 1024), (33, 2112, 4096),
                                   # few enough columns, but more tokens than two workgroups on a compute unit have LDS for
                                   (17, 2048, 8192), (24, 2048, 8192), (32, 2048, 8192), (32, 1600, 8192), (17, 2048, 6144), (25, 1536, 4096),
                                   (31, 1088, 2048), (30, 1536, 5056), (33, 512, 2048), (64, 512, 2048), (49, 448, 1536), (41, 64, 128),
                                   (33, 1024, 4096), (48, 576, 3648)])
def test_layers_beyond_its_sizes_take_two_launches(T, d, F):
    assert not L.lib().stem_route_one_launch(d, F, ctypes.c_int64(T))
    s = _layer(T, d, F, 300, 5)
    ctx = L.stem_create(d, F, 300, L.STEM_BF16, T, 0)
    y = _call(ctx, s, torch.empty_like(s["x"]))
    L.stem_sync_status(ctx)
    f = {k: inputs.to_f64(v) for k, v in s.items() if k != "ids"}
    ref = O.ffn_forward(f["x"], s["ids"].cpu().numpy(), f["Wg"], f["Wd"], f["E"])[0] + f["r"]
    assert (np.abs(inputs.to_f64(y) - ref) <= _bound(s, ref)).all()
    ctx.close()


@pytest.mark.parametrize("over", ["W_down", "y"])
def test_saved_activations_over_what_two_launches_read_later(over):
    """Two launches have stored H (and G) when W_down is read and y stored; one launch has not, and leaves the call to them."""
    T, d, F, V = 8, 64, 64, 50
    s = _layer(T, d, F, V, 9)
    ctx = L.stem_create(d, F, V, L.STEM_BF16, T, 0)
    H = torch.empty(T, F, dtype=torch.bfloat16, device=DEV)
    y = torch.empty_like(s["x"])
    L.stem_ffn_forward(ctx, s["x"], s["ids"], s["Wg"], s["Wd"], s["E"], y, None, H)
    wd, out, G = s["Wd"].clone(), torch.empty_like(y), torch.empty_like(H)
    if over == "W_down":       # its first rows become G (T x F values)
        G = wd.view(-1)[:T * F].view(T, F)
    if over == "y":            # (d = F) y is stored last
        G = out
    L.stem_ffn_forward(ctx, s["x"], s["ids"], s["Wg"], wd, s["E"], out, G, None)
    L.stem_sync_status(ctx)
    f = {k: inputs.to_f64(v) for k, v in s.items() if k != "ids"}
    want = inputs.to_f64(H) @ inputs.to_f64(wd).T
    assert Hn.max_rel(out.float().cpu(), want) < 1e-2
    ctx.close()
