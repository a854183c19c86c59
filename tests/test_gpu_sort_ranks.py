"""The sort of up to 8192 ids by counting ranks, or beyond 2048 by buckets of the vocabulary, against the oracle: sizes about their workgroups
and keys per thread, vocabularies about the bitmap's size, and outputs that lie over the ids."""
import numpy as np
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

DEV = "cuda:0"

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,route", [
    (7, 40, Hn.SORT_ONE_1024), (8, 33, Hn.SORT_ONE_1024), (9, 32, Hn.SORT_ONE_1024), (1023, 1 << 18, Hn.SORT_ONE_1024),
    (1024, 65, Hn.SORT_ONE_1024), (1025, 1 << 18, Hn.SORT_ONE_4096), (2047, 257, Hn.SORT_ONE_4096), (2048, 128256, Hn.SORT_ONE_4096),
    (2049, 31, Hn.SORT_ONE_4096), (4096, 1 << 18, Hn.SORT_ONE_4096), (4097, 1 << 18, Hn.SORT_RUNS_1024), (8191, 8193, Hn.SORT_RUNS_1024),
    (8192, 1 << 18, Hn.SORT_RUNS_1024),
    # one id more than the bitmap holds: the kernels for larger vocabularies
    (1000, (1 << 18) + 1, Hn.SORT_ONE_1024), (3000, (1 << 18) + 1, Hn.SORT_ONE_4096), (8192, (1 << 18) + 1, Hn.SORT_RUNS_1024),
    (8193, 1 << 18, Hn.SORT_RUNS_1024),
])
def test_ranks_by_counting(T, V, route):
    """`route`: what sorts where an output lies over the ids, or beyond the bitmap's vocabularies."""
    assert Hn.route_sort(T, V) == route
    rng = np.random.default_rng(91)
    mixed = inputs.zipf_ids(T, V, seed=91)
    mixed[T // 2:] = rng.integers(0, V, T - T // 2)
    mixed[0], mixed[-1] = V - 1, 0
    batches = [mixed, np.full(T, V - 1, np.int32), np.arange(T - 1, -1, -1, dtype=np.int32) % V]
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    for ids in batches:
        ids = ids.astype(np.int32)
        dev = torch.from_numpy(ids).to(DEV)
        eg = Hn.hip_embed_grad(ctx, dev, None, V, with_rows=False)
        Hn.check_integers(eg, ids)
        lie = {k: eg[k].data_ptr() for k in ("sorted_ids", "perm", "uniq_ids", "seg_offsets", "n_uniq")}
        assert Hn.route_sort_ranks(T, V, ids=dev.data_ptr(), **lie) == (T <= 2048 and V <= 1 << 18)
        assert Hn.route_sort_buckets(T, V, ids=dev.data_ptr(), **lie) == (T > 2048 and V <= 1 << 18)
        # an output over the ids, and one that begins at their last
        for name in ("sorted_ids", "perm", "uniq_ids"):
            room = torch.zeros(2 * T, dtype=torch.int32, device=DEV)
            for at in (0, T - 1):
                room[:T] = torch.from_numpy(ids).to(DEV)
                out = dict(eg)
                out[name] = room[at:at + eg[name].shape[0]]
                L.stem_embed_grad(ctx, room[:T], None, out["sorted_ids"], out["perm"], out["uniq_ids"], out["seg_offsets"],
                                  out["n_uniq"], None, T=T)
                Hn.check_integers(out, ids)
    L.stem_sync_status(ctx)
    ctx.close()


@pytest.mark.parametrize("T", [700, 1500, 3000, 6000])
def test_ids_outside_the_table_count_as_the_clamped_ones(T):
    V = 300
    ids = inputs.zipf_ids(T, V, seed=92)
    ids[[0, 5, T // 2, T - 1]] = [V, -1, 2 ** 31 - 1, -2 ** 31]
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    eg = Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), None, V, with_rows=False)
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    Hn.check_integers(eg, np.clip(ids.astype(np.int64), 0, V - 1).astype(np.int32))
    ctx.close()


@pytest.mark.parametrize("T,V", [(7, 40), (1000, 300), (1000, 5000), (4096, 1 << 18), (4097, 1 << 18), (8192, 128256)])
def test_outputs_over_the_ids_and_over_each_other(T, V):
    """Every output over the ids, whole and by one element, and the sorted ids where the distinct ones go (up to 4096 ids: beyond, the
    runs' kernels number the distinct ids while others still read the sorted ones).  What a call does not write stays as it was."""
    ids = inputs.zipf_ids(T, V, seed=93).astype(np.int32)
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    cap = min(T, V)
    size = dict(sorted_ids=T, perm=T, uniq_ids=cap, seg_offsets=cap + 1, n_uniq=1)
    U = len(np.unique(ids))

    def call(over):
        out = {k: torch.full((n,), -9, dtype=torch.int32, device=DEV) for k, n in size.items()}
        room = torch.full((2 * T + 2,), -9, dtype=torch.int32, device=DEV)
        room[:T] = torch.from_numpy(ids).to(DEV)
        for name, at in over.items():
            out[name] = out[at] if isinstance(at, str) else room[at:at + size[name]]
        lie = {k: v.data_ptr() for k, v in out.items()}
        ranks, buckets = (f(T, V, ids=room.data_ptr(), **lie) for f in (Hn.route_sort_ranks, Hn.route_sort_buckets))
        assert (ranks, buckets) == (not over and T <= 2048, not over and T > 2048)
        L.stem_embed_grad(ctx, room[:T], None, out["sorted_ids"], out["perm"], out["uniq_ids"], out["seg_offsets"], out["n_uniq"], None, T=T)
        return out

    whole = call({})
    Hn.check_integers(whole, ids)
    assert bool((whole["uniq_ids"][U:] == -9).all()) and bool((whole["seg_offsets"][U + 1:] == -9).all())
    for name in size:
        for at in (0, T - 1):
            Hn.check_integers(call({name: at}), ids)
    if T <= 4096 and T <= V:
        out = call({"sorted_ids": "uniq_ids"})
        assert int(out["n_uniq"].item()) == U
        for name, n in (("uniq_ids", U), ("seg_offsets", U + 1), ("perm", T)):
            assert torch.equal(out[name][:n], whole[name][:n])
    L.stem_sync_status(ctx)
    ctx.close()
