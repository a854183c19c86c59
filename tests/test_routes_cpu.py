"""CPU-only: the rules that choose a call's kernels, asked through the library itself."""
import ctypes
import random

import pytest

from paper_2601_10639_amd import stemlib as L
from tests.harness import DECODE, EPI_BF16, EPI_F32, EPI_GATE, FEW_ROW, TILES, route_forward, route_gate_up_together, route_sort_buckets, route_sort_ranks, route_sort_sum, route_tiles as tiles, route_weight_grads, route_weight_grads_apart


def test_no_k_slice_is_empty():
    """Every slice of a split product has a K tile: 64-wide K tiles, dealt to the slices (of each operand pair) in runs
    of equal length."""
    rng = random.Random(1)
    split = 0
    for _ in range(20000):
        M, N = rng.choice([rng.randint(1, 3000), 64 * rng.randint(1, 40)]), 64 * rng.randint(1, 64)
        K, ops, epi = 64 * rng.randint(1, 140), rng.choice([1, 2]), rng.choice([EPI_BF16, EPI_F32])
        if epi == EPI_F32:
            K, ops = rng.randint(1, 9000), 1
        _, _, _, ks = tiles(M, N, K, ops, epi)
        if ks == 1:
            continue
        split += 1
        assert ks % ops == 0 and 4 * M * N * ks <= 64 << 20, (M, N, K, ops, epi, ks)
        nk, per_pair = -(-K // 64), ks // ops
        assert (per_pair - 1) * -(-nk // per_pair) < nk, (M, N, K, ops, epi, ks)
    assert split > 1000
    assert tiles(600, 512, 33 * 64)[3] == 7      # 33 K tiles in runs of 5


@pytest.mark.parametrize("product,want", [
    # 256x256 tiles that end in part of a round, against whole rounds of 256x128 ones: us, 256x256 / 256x128
    ((16384, 3328, 1280, 1, EPI_GATE), (256, 256, 1)),      # 166 / 180
    ((24000, 1536, 5120, 2, EPI_BF16), (256, 256, 1)),      # 646 / 732
    ((49152, 512, 1536, 1, EPI_BF16), (256, 256, 1)),       # 83 / 99
    ((1536, 5120, 16384, 1, EPI_F32), (256, 256, 2)),       # 214 / 245
    # and where the smaller tiles are the better ones
    ((1999, 2048, 8192, 1, EPI_BF16), (128, 128, 1)),       # 146 / 92 / 70 for 128x128
    ((4096, 2048, 8192, 1, EPI_BF16), (256, 128, 1)),       # 165 / 114
])
def test_tiling_of_products_that_were_measured_on_each(product, want):
    assert tiles(*product)[1:] == want


@pytest.mark.parametrize("T,d,F,n,together", [
    # as many rounds either way: backward, us, launches of their own / one launch
    (6773, 1344, 5312, 3, False),      # 601 / 617
    (7961, 1472, 3840, 3, False),      # 542 / 568
    (21592, 1792, 7104, 2, False),     # 1915 / 1952
    (24323, 1984, 5696, 2, False),     # 1924 / 1945
    (1999, 2048, 8192, 2, True),       # 271 / 270
    (1013, 1920, 6400, 2, True),       # 130 / 126
    # fewer rounds or slices
    (16384, 1024, 4096, 2, True),      # 541 / 508
    (4096, 1024, 4096, 3, True),       # 225 / 211
    (395, 576, 1728, 2, True),         # 36 / 30
])
def test_weight_gradients_share_a_launch_where_that_was_measured_shorter(T, d, F, n, together):
    assert bool(route_weight_grads(T, d, F, n, min(64 << 20, 32 * d * max(T, F)))[0]) == together


def test_weight_gradients_over_buffers_that_are_read_before_them_do_not_share_a_launch():
    T, d, F = 700, 192, 576
    size = dict(dy=T * d * 2, H=T * F * 2, dx=T * d * 2, W_gate=F * d * 2, W_up=F * d * 2, dV=T * F * 2, dW_gate=F * d * 4, dW_up=F * d * 4)
    for up in (False, True):
        names = [k for k in size if up or k not in ("W_up", "dV", "dW_up")]
        lie = {k: (i + 1) << 24 for i, k in enumerate(names)}
        assert route_weight_grads_apart(T, d, F, **lie)
        for grad in ("dW_gate", "dW_up") if up else ("dW_gate",):
            for over in set(names) - {grad, "dx", "dW_gate", "dW_up"}:
                before_dx = over in ("dy", "H")   # read by dW_down; the others by dx, and dV by dW_up
                for with_dx in (True, False):
                    q = {**lie, "dx": lie["dx"] if with_dx else None}
                    refused = before_dx or with_dx or (over == "dV" and grad == "dW_gate")
                    for at, shares in ((lie[over] - size[grad], True), (lie[over] - size[grad] + 16, not refused),
                                       (lie[over] + size[over] - 16, not refused), (lie[over] + size[over], True)):
                        assert route_weight_grads_apart(T, d, F, **{**q, grad: at}) == shares, (up, grad, over, with_dx, at)


@pytest.mark.parametrize("T,d,F,dtype,rows,streams", [
    # three contexts in turn, one copy stream / two in turn, us
    (2000, 512, 1536, L.STEM_BF16, 845, 2),         # 65 / 55
    (4096, 1024, 4096, L.STEM_BF16, 1421, 2),       # 227 / 209
    (65536, 1024, 4096, L.STEM_BF16, 10913, 2),     # 1691 / 1643
    (16384, 2048, 8192, L.STEM_BF16, 4677, 2),      # 1404 / 1357
    (12668, 1472, 5248, L.STEM_BF16, 2421, 1),      # 495 / 515: the products weigh as much as the rows
    (16384, 2048, 8192, L.STEM_BF16, 3804, 1),      # 1170 / 1240
    (40000, 2048, 8192, L.STEM_BF16, 9189, 1),      # 2836 / 3013
    (65536, 2048, 8192, L.STEM_BF16, 51237, 1),     # long
    (700, 2048, 8192, L.STEM_BF16, 390, 1),         # 124 / 146
    (850, 2048, 6144, L.STEM_BF16, 450, 1),         # 110 / 119
    (850, 1728, 5824, L.STEM_BF16, 450, 2),         # 107 / 106
    (1000, 256, 1024, L.STEM_F32, 407, 2),          # 55 / 45
    (2000, 512, 2048, L.STEM_F32, 670, 1),          # 131 / 149
])
def test_host_table_calls_that_share_the_link_where_that_was_measured_shorter(T, d, F, dtype, rows, streams):
    assert L.lib().stem_route_copy_streams(d, F, dtype, ctypes.c_int64(T), ctypes.c_int64(rows)) == streams


@pytest.mark.parametrize("T,d,F,gate,touched", [
    (111, 1024, 4096, DECODE, False),
    (112, 1024, 4096, DECODE, True),
    (128, 2048, 8192, DECODE, True),
    (192, 2048, 8192, FEW_ROW, False),
    (384, 1536, 5120, FEW_ROW, True),
    (450, 1280, 5120, TILES, False),      # other kernels' arguments stand there for the tile kernel
    (512, 1536, 5120, TILES, False),
    (513, 1024, 4096, TILES, False),
])
def test_gate_products_that_touch_the_down_products_weights(T, d, F, gate, touched):
    assert route_forward(T, d, F)[0][0] == gate
    assert L.lib().stem_route_touch_bytes(d, F, ctypes.c_int64(T)) == (2 * d * F if touched else 0)


@pytest.mark.parametrize("table", [False, True])
def test_gate_and_up_product_over_buffers_that_the_other_reads_do_not_share_a_launch(table):
    T, d, F, V = 300, 256, 832, 500
    TF = T * F * 2
    size = dict(W_up=F * d * 2, E=V * F * 2, ids=T * 4, G=TF, Up=TF, H=TF)
    lie = {k: (i + 1) << 24 for i, k in enumerate(size) if table or k not in ("E", "ids")}

    def share(**at):
        return route_gate_up_together(T, d, F, V if table else 0, **{**lie, **at})

    assert share() and share(G=None) and share(G=lie["Up"]) and share(H=lie["Up"]) and share(G=lie["H"])
    for out, over in [(o, i) for o in ("G", "Up", "H") for i in lie if i != o and (o == "Up" or i in ("W_up", "Up"))]:
        if out == "Up" and over in ("G", "H"):
            continue                                       # asked as G and H over Up
        at = lie[over]
        assert share(**{out: at - TF}) and share(**{out: at + size[over]}), (out, over)
        for p in (at - TF + 16, at + size[over] - 16, *([at] if over != "Up" else [])):
            assert not share(**{out: p}), (out, over, p - at)
    # what one after the other did not keep either: G and H over the table, the ids and each other
    if table:
        assert share(G=lie["E"]) and share(H=lie["ids"])


@pytest.mark.parametrize("T,V,route", [(7, 40, route_sort_ranks), (1000, 300, route_sort_ranks), (2048, 1 << 18, route_sort_ranks),
                                       (2049, 300, route_sort_buckets), (4096, 1 << 18, route_sort_buckets), (16384, 128256, route_sort_buckets)])
def test_ranks_are_counted_and_buckets_sorted_where_no_two_buffers_of_the_sort_overlap(T, V, route):
    cap = min(T, V)
    size = dict(ids=T, sorted_ids=T, perm=T, uniq_ids=cap, seg_offsets=cap + 1, n_uniq=1, seg_of=T)
    lie = {k: (i + 1) << 24 for i, k in enumerate(size)}
    assert route(T, V, **lie) and not route(T, (1 << 18) + 1, **lie)
    assert route_sort_ranks(2048, V, **lie) and not route_sort_ranks(2049, V, **lie)
    assert not route_sort_buckets(2048, V, **lie) and route_sort_buckets(2049, V, **lie)
    assert route_sort_buckets(16384, V, **lie) and not route_sort_buckets(16385, V, **lie)
    for a in size:
        for b in size:
            if a == b:
                continue
            for at, ranks in ((lie[b] - 4 * size[a], True), (lie[b] - 4 * size[a] + 4, False), (lie[b], False),
                              (lie[b] + 4 * size[b] - 4, False), (lie[b] + 4 * size[b], True)):
                assert route(T, V, **{**lie, a: at}) == ranks, (a, b, at - lie[b])


@pytest.mark.parametrize("bf16,T,V,F", [(True, 7, 40, 64), (False, 1000, 300, 1024), (True, 512, 1 << 17, 8192), (True, 2048, 128256, 8192)])
def test_sort_and_sums_share_a_launch_where_no_two_of_their_buffers_overlap(bf16, T, V, F):
    cap, es = min(T, V), 2 if bf16 else 4
    ints = dict(ids=T, sorted_ids=T, perm=T, uniq_ids=cap, seg_offsets=cap + 1, n_uniq=1, seg_of=T)
    size = dict(dU=T * F * es, dE_rows=cap * F * 4, **{k: 4 * n for k, n in ints.items()})
    lie = {k: (i + 1) << 28 for i, k in enumerate(size)}
    share = lambda **over: route_sort_sum(bf16, T, V, F, **{**lie, **over})
    assert share() and not share(dU=0)
    assert not route_sort_sum(bf16, T, (1 << 17) + 1, F, **lie) and not route_sort_sum(bf16, 2049, V, F, **lie)
    assert not route_sort_sum(bf16, T, V, 1 << 23, **lie)
    for a in size:
        for b in size:
            if a == b:
                continue
            for at, one in ((lie[b] - size[a], True), (lie[b] - size[a] + 4, False), (lie[b], False), (lie[b] + size[b] - 4, False),
                            (lie[b] + size[b], True)):
                assert share(**{a: at}) == one, (a, b, at - lie[b])


@pytest.mark.parametrize("T,d,F", [(1, 64, 64), (24, 1024, 4096)])
def test_saved_activations_beside_the_layer_in_one_launch(T, d, F):
    size = dict(G=T * F * 2, H=T * F * 2, W_down=F * d * 2, residual=T * d * 2, y=T * d * 2)
    lie = {k: (i + 1) << 28 for i, k in enumerate(size)}
    apart = lambda **over: bool(L.lib().stem_route_one_launch_apart(d, F, ctypes.c_int64(T), *[ctypes.c_void_p({**lie, **over}[k]) for k in size]))
    assert apart() and apart(G=None, H=None) and apart(G=lie["H"]) and apart(residual=lie["y"]) and apart(residual=lie["W_down"])
    for a in ("G", "H"):
        for b in ("W_down", "residual", "y"):
            for at, ok in ((lie[b] - size[a], True), (lie[b] - size[a] + 2, False), (lie[b], False), (lie[b] + size[b] - 2, False),
                           (lie[b] + size[b], True)):
                assert apart(**{a: at}) == ok, (a, b, at - lie[b])


def test_sizes_of_the_layer_in_one_launch():
    one = lambda T, d, F: bool(L.lib().stem_route_one_launch(d, F, ctypes.c_int64(T)))
    assert one(1, 64, 64) and not one(0, 64, 64) and not one(1, 2112, 64) and not one(1, 64, 8256)
    for d, most in ((64, 32), (512, 32), (576, 32), (1024, 32), (1088, 24), (1536, 24), (1600, 16), (2048, 16)):
        for F in (64, 3648, 4096, 8192):
            assert all(one(T, d, F) == (T <= most) for T in range(1, 66)), (d, F)


def test_launch_numbers_of_the_layer_in_one_launch_are_never_what_an_idle_claim_holds():
    """A workgroup looks for shares that were given up until no claim holds the launch's number, and idle claims hold 0."""
    after = L.lib().stem_next_launch
    after.restype = ctypes.c_uint32
    number = lambda last: after(ctypes.c_uint32(last))
    most = 2 ** 32 - 1
    assert [number(n) for n in (0, 1, 2 ** 31 - 1, 2 ** 31, most - 1)] == [1, 2, 2 ** 31, 2 ** 31 + 1, most] and number(most) == 1
    for last in (0, most - 4):
        seen = [last]
        for _ in range(8):
            seen.append(number(seen[-1]))
            claims, looks = [0] * 256, 0
            while seen[-1] in claims and looks < 300:      # (taken: back to 0)
                claims[claims.index(seen[-1])] = 0
                looks += 1
            assert looks == 0 and seen[-1] != 0
        assert len(set(seen)) == len(seen)                 # no number is left of a launch before
