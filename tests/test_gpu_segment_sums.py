"""Table gradient of small batches, summed in one launch, at the sizes where its runs and slabs can go wrong."""
import numpy as np
import pytest
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _ids(kind, T, V):
    rng = np.random.default_rng(T)
    if kind == "equal":
        return np.full(T, V - 1, np.int32)
    if kind == "distinct":
        return rng.permutation(V)[:T].astype(np.int32)
    if kind == "runs":   # 15, 16, 17, 33 and 64 rows (a round of loads, one more row than that, one more than two), then singles
        out = np.concatenate([np.full(n, 3 * i, np.int32) for i, n in enumerate((15, 16, 17, 33, 64))])
        return rng.permutation(np.concatenate([out, 1000 + np.arange(T - out.size)]).astype(np.int32))
    return inputs.zipf_ids(T, V, seed=7)


@pytest.mark.parametrize("dtype,T,F,kind", [
    ("f32", 1, 4, "equal"), ("f32", 128, 256, "zipf"), ("f32", 1024, 260, "equal"), ("f32", 1024, 2048, "zipf"),
    ("f32", 500, 516, "runs"), ("f32", 1024, 64, "distinct"), ("f32", 1024, 2052, "zipf"), ("f32", 1025, 256, "runs"),
    ("bf16", 1, 64, "equal"), ("bf16", 130, 8192, "zipf"), ("bf16", 1024, 576, "equal"), ("bf16", 512, 8192, "runs"),
    ("bf16", 513, 8192, "zipf"), ("bf16", 300, 576, "distinct"), ("bf16", 1000, 4160, "zipf"),
])
def test_rows_of_small_batches(dtype, T, F, kind):
    V = 3000
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ids = _ids(kind, T, V)
    dU = inputs.normal((T, F), 1.0, 11, dt, DEV)
    ctx = Hn.make_ctx(inputs.StemShape("runs", 64, F, V, 1, T, dtype), T)
    a, b = (Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), dU, V) for _ in range(2))
    L.stem_sync_status(ctx)
    U = Hn.check_integers(a, ids)
    x = inputs.to_f64(dU)
    ref, size = O.embed_grad(ids, x)["dE_rows"], O.embed_grad(ids, np.abs(x))["dE_rows"]
    n = np.unique(ids, return_counts=True)[1]
    got = a["dE_rows"][:U].cpu().numpy().astype(np.float64)
    # a sum of n terms, in chunks or stretches whichever way, is off by at most n - 1 roundings of at most the sum of magnitudes
    assert (np.abs(got - ref) <= n[:, None] * 2.0 ** -24 * size + 1e-30).all()
    assert torch.equal(a["dE_rows"][:U], b["dE_rows"][:U])
    ctx.close()


@pytest.mark.parametrize("dtype,F,lengths", [
    ("f32", 260, (17, 64, 65, 128, 129, 256, 257)),   # the edges of a run's split over wavefronts and workgroups
    ("f32", 1028, (512, 511)), ("f32", 64, (513, 500)), ("f32", 2048, (1024,)),
    ("bf16", 576, (17, 64, 65, 128, 129, 256, 257)), ("bf16", 4160, (512,)), ("bf16", 64, (513, 500)), ("bf16", 512, (1024,)),
])
def test_long_runs_of_small_batches_are_not_summed_in_one_chain(dtype, F, lengths):
    V = 3000
    ids = np.repeat(np.arange(len(lengths), dtype=np.int32) * 7, lengths)
    T = ids.size
    ids = np.random.default_rng(T).permutation(ids)
    if dtype == "bf16":
        dU = inputs.normal((T, F), 1.0, 13, torch.bfloat16, DEV)
    else:   # numbers that a chain of additions rounds the same way each time: 1024 of them in four stretches lose 62 units of 2^-24
        dU = (1.0 + 2.0 ** -(8.0 + torch.arange(F, device=DEV) % 15) - 2.0 ** -23).float().repeat(T, 1)
    ctx = Hn.make_ctx(inputs.StemShape("long-runs", 64, F, V, 1, T, dtype), T)
    a, b = (Hn.hip_embed_grad(ctx, torch.from_numpy(ids).to(DEV), dU, V) for _ in range(2))
    L.stem_sync_status(ctx)
    U = Hn.check_integers(a, ids)
    x = inputs.to_f64(dU)
    ref, size = O.embed_grad(ids, x)["dE_rows"], O.embed_grad(ids, np.abs(x))["dE_rows"]
    got = a["dE_rows"][:U].cpu().numpy().astype(np.float64)
    # 3 additions in a group of four rows, 7 of groups of four, 7 of row groups in a wavefront, 3 of wavefronts
    assert (np.abs(got - ref) <= 20 * 2.0 ** -24 * size).all(), float((np.abs(got - ref) / size).max() * 2.0 ** 24)
    assert torch.equal(a["dE_rows"][:U], b["dE_rows"][:U])
    ctx.close()
