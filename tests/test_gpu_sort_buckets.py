"""The sort of 2049 to 16384 ids by buckets of the vocabulary, against the oracle: sizes about its chunks, vocabularies about its buckets."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _batches(T, V):
    rng = np.random.default_rng(T + V)
    mixed = inputs.zipf_ids(T, V, seed=91)
    mixed[T // 2:] = rng.integers(0, V, T - T // 2)
    mixed[0], mixed[-1] = V - 1, 0
    one_bucket = rng.integers(0, min(32, V), T)                    # a bucket's wavefronts with many rounds each
    edges = np.array([i for k in range(0, V, 32) for i in (k, k + 31) if i < V])
    return [mixed, np.full(T, V - 1), np.full(T, 0), np.arange(T - 1, -1, -1) % V, one_bucket, rng.choice(edges, T), rng.permutation(np.arange(T) % V)]


@pytest.mark.parametrize("T,V,buckets", [
    (2049, 31, True), (2049, 1 << 18, True), (4096, 33, True), (4096, 50304, True), (4097, 8193, True), (8192, 128256, True), (8193, 1000, True),
    (16383, 257, True), (16384, 1, True), (16384, 50304, True), (16384, 1 << 18, True),
    (2048, 50304, False), (16385, 50304, False), (5000, (1 << 18) + 1, False),
])
def test_buckets(T, V, buckets):
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    for ids in _batches(T, V):
        ids = ids.astype(np.int32)
        dev = torch.from_numpy(ids).to(DEV)
        eg = Hn.hip_embed_grad(ctx, dev, None, V, with_rows=False)
        at = {k: v.data_ptr() for k, v in eg.items() if v is not None and k != "dE_rows"}
        assert Hn.route_sort_buckets(T, V, ids=dev.data_ptr(), **at) == buckets
        U = Hn.check_integers(eg, ids)
        if T <= 5000:   # the run index: sums of one column of ones
            dU = torch.ones(T, 64, dtype=torch.bfloat16, device=DEV)
            rows = torch.empty(min(T, V), 64, dtype=torch.float32, device=DEV)
            L.stem_embed_grad_presorted(ctx, dU, eg["perm"], eg["seg_offsets"], rows, T=T)
            assert np.array_equal(rows[:U, 0].cpu().numpy(), np.unique(ids, return_counts=True)[1])
    L.stem_sync_status(ctx)
    ctx.close()


def test_ids_outside_the_table_count_as_the_clamped_ones():
    T, V = 5000, 300
    ids = inputs.zipf_ids(T, V, seed=92)
    ids[[0, 5, T // 2, T - 1]] = [V, -1, 2 ** 31 - 1, -2 ** 31]
    ctx = L.stem_create(64, 64, V, L.STEM_BF16, T, 0)
    eg = Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), None, V, with_rows=False)
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    Hn.check_integers(eg, np.clip(ids.astype(np.int64), 0, V - 1).astype(np.int32))
    ctx.close()
