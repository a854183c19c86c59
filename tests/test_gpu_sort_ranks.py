"""The sort of up to 8192 ids by counting ranks, against the oracle: sizes about its workgroups and its keys per thread, vocabularies about
its bitmap's size, and outputs that lie over the ids."""
import numpy as np
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

DEV = "cuda:0"
RANKS_8192 = 5

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,route", [
    (7, 40, Hn.SORT_ONE_1024), (8, 33, Hn.SORT_ONE_1024), (9, 32, Hn.SORT_ONE_1024), (1023, 1 << 18, Hn.SORT_ONE_1024),
    (1024, 65, Hn.SORT_ONE_1024), (1025, 1 << 18, Hn.SORT_ONE_4096), (2047, 257, Hn.SORT_ONE_4096), (2048, 128256, Hn.SORT_ONE_4096),
    (2049, 31, Hn.SORT_ONE_4096), (4096, 1 << 18, Hn.SORT_ONE_4096), (4097, 1 << 18, RANKS_8192), (8191, 8193, RANKS_8192),
    (8192, 1 << 18, RANKS_8192),
    # one id more than the bitmap holds: the kernels for larger vocabularies
    (1000, (1 << 18) + 1, Hn.SORT_ONE_1024), (3000, (1 << 18) + 1, Hn.SORT_ONE_4096), (8192, (1 << 18) + 1, Hn.SORT_RUNS_1024),
    (8193, 1 << 18, Hn.SORT_RUNS_1024),
])
def test_ranks_by_counting(T, V, route):
    assert Hn.route_sort(T, V) == route
    rng = np.random.default_rng(91)
    mixed = inputs.zipf_ids(T, V, seed=91)
    mixed[T // 2:] = rng.integers(0, V, T - T // 2)
    mixed[0], mixed[-1] = V - 1, 0
    batches = [mixed, np.full(T, V - 1, np.int32), np.arange(T - 1, -1, -1, dtype=np.int32) % V]
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    for ids in batches:
        ids = ids.astype(np.int32)
        eg = Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), None, V, with_rows=False)
        Hn.check_integers(eg, ids)
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
