"""Sort and row sums of a small batch in one launch: the oracle's integers, and the bits that the two launches give."""
import numpy as np
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _batches(T, V):
    rng = np.random.default_rng(T)
    mixed = inputs.zipf_ids(T, V, seed=91)
    mixed[T // 2:] = rng.integers(0, V, T - T // 2)
    mixed[0], mixed[-1] = V - 1, 0
    runs = np.repeat(np.arange(7), (16, 17, 64, 65, 128, 129, 257))[:T]   # the edges of a run's split over wavefronts and workgroups
    runs = np.concatenate([runs * 31 % V, rng.integers(0, V, T - runs.size)])
    return [mixed, np.full(T, V - 1), np.arange(T - 1, -1, -1) % V, rng.permutation(runs)]


@pytest.mark.parametrize("dtype,T,V,F,one", [
    ("f32", 1, 40, 4, True), ("f32", 64, 33, 256, True), ("f32", 65, 32, 260, True), ("f32", 256, 1 << 17, 64, True),
    ("f32", 257, 1000, 516, True), ("f32", 1024, 1 << 17, 1028, True), ("f32", 1023, 8000, 2048, True),
    ("bf16", 1, 64, 64, True), ("bf16", 63, 31, 512, True), ("bf16", 255, 128256, 576, True), ("bf16", 512, 8192, 8192, True),
    ("bf16", 1024, 3000, 4096, True), ("bf16", 1025, 3000, 512, True), ("f32", 2048, 1000, 260, True), ("bf16", 2047, 128256, 8192, True),
    # the edges of bands and teams
    ("bf16", 256, 3000, 8256, True), ("bf16", 257, 3000, 8256, True), ("bf16", 513, 3000, 8256, True), ("f32", 512, 3000, 1028, True),
    # past the vocabulary's bitmap, the tokens and the workgroups: two launches
    ("f32", 300, (1 << 17) + 1, 256, False), ("bf16", 1999, (1 << 17) + 1, 576, False), ("f32", 2049, 1000, 256, False),
    ("f32", 2048, 1000, 16388, False),
])
def test_sort_and_sums_in_one_launch(dtype, T, V, F, one):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dU = inputs.normal((T, F), 1.0, 11, dt, DEV)
    ctx = Hn.make_ctx(inputs.StemShape("small", 64, F, V, 1, T, dtype), T)
    for ids in _batches(T, V):
        ids = ids.astype(np.int32)
        dev_ids = torch.from_numpy(ids).to(DEV)
        eg = Hn.hip_embed_grad(ctx, dev_ids, dU, V)
        at = {k: v.data_ptr() for k, v in eg.items()}
        assert Hn.route_sort_sum(dtype == "bf16", T, V, F, ids=dev_ids.data_ptr(), dU=dU.data_ptr(), **at) == one
        U = Hn.check_integers(eg, ids)
        again = torch.empty_like(eg["dE_rows"])
        L.stem_embed_grad_presorted(ctx, dU, eg["perm"], eg["seg_offsets"], again, T=T)   # with the run index of that call
        assert torch.equal(eg["dE_rows"][:U], again[:U])
        two = Hn.hip_embed_grad(ctx, dev_ids, None, V, with_rows=False)
        L.stem_embed_grad_presorted(ctx, dU, two["perm"], two["seg_offsets"], again, T=T)
        assert torch.equal(eg["dE_rows"][:U], again[:U])
    L.stem_sync_status(ctx)
    ctx.close()


def test_ids_outside_the_table_count_as_the_clamped_ones():
    T, V, F = 700, 300, 256
    ids = inputs.zipf_ids(T, V, seed=92)
    ids[[0, 5, T // 2, T - 1]] = [V, -1, 2 ** 31 - 1, -2 ** 31]
    clamped = np.clip(ids.astype(np.int64), 0, V - 1).astype(np.int32)
    dU = inputs.normal((T, F), 1.0, 11, torch.float32, DEV)
    ctx = Hn.make_ctx(inputs.StemShape("small", 64, F, V, 1, T, "f32"), T)
    eg = Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), dU, V)
    with pytest.raises(L.StemError) as e:
        L.stem_sync_status(ctx)
    assert e.value.status == L.STEM_ERR_ID_RANGE
    U = Hn.check_integers(eg, clamped)
    ref = Hn.hip_embed_grad(ctx, torch.from_numpy(clamped).to(DEV), dU, V)
    L.stem_sync_status(ctx)
    assert torch.equal(eg["dE_rows"][:U], ref["dE_rows"][:U])
    ctx.close()
