"""Copy of a batch's distinct rows from pinned host memory, at the sizes where its pieces of 1 KB can go wrong: rows of one
vector, of whole pieces, of a piece and a vector; fewer pieces than wavefronts, and more than they look up at a time."""
import numpy as np
import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,F", [("f32", 4), ("f32", 256), ("f32", 260), ("bf16", 64), ("bf16", 512), ("bf16", 8256)])
@pytest.mark.parametrize("n", [1, 65, 5000])
def test_rows_arrive_whole_and_nothing_else_is_written(dtype, F, n):
    T, V = n, 6000
    if F == 8256 and n == 5000:
        T = 400                              # 6800 pieces
    shape = inputs.StemShape("rows", 64, F, V, 1, T, dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ids = np.random.default_rng(n + F).permutation(V)[:T].astype(np.int32)
    E_host = inputs.normal((V, F), 1.0, 5, dt, "cpu").pin_memory()
    E_compact = torch.full((T + 3, F), 7.0, dtype=dt, device=DEV)
    remap = torch.empty(T, dtype=torch.int32, device=DEV)
    ctx = Hn.make_ctx(shape, T)
    rows, _ = L.stem_prefetch_rows(ctx, E_host, torch.from_numpy(ids), E_compact, remap)
    torch.cuda.synchronize()
    assert rows == T
    assert torch.equal(E_compact[:T].cpu(), E_host[torch.from_numpy(np.sort(ids)).long()])
    assert bool((E_compact[T:] == 7.0).all())
    ctx.close()


@pytest.mark.parametrize("T,max_tokens,V", [(1, 7, 5), (255, 70001, 300), (257, 70001, 300), (66001, 70001, 300), (300001, 300003, 1000)])
def test_remap_of_long_batches_and_of_batches_without_a_miss(T, max_tokens, V):
    """Lists shorter than the context's arrays, and longer than one sweep of the kernel that brings them."""
    F = 4
    shape = inputs.StemShape("lists", 64, F, V, 1, max_tokens, "f32")
    ids = np.random.default_rng(T).integers(0, V, T).astype(np.int32)
    distinct, want = np.unique(ids, return_inverse=True)
    E_host = inputs.normal((V, F), 1.0, 6, torch.float32, "cpu").pin_memory()
    ctx = Hn.make_ctx(shape, max_tokens)
    E_compact = torch.empty(V, F, dtype=torch.float32, device=DEV)
    remap = torch.full((T + 3,), -7, dtype=torch.int32, device=DEV)
    n, _ = L.stem_prefetch_rows(ctx, E_host, torch.from_numpy(ids), E_compact, remap, T=T)
    torch.cuda.synchronize()
    assert n == distinct.size
    np.testing.assert_array_equal(remap[:T].cpu().numpy(), want)
    assert bool((remap[T:] == -7).all())
    assert torch.equal(E_compact[:n].cpu(), E_host[torch.from_numpy(distinct).long()])
    L.stem_cache_init(ctx, V)
    E_dev = torch.empty(2 * V, F, dtype=torch.float32, device=DEV)
    for batch in range(2):   # the second finds every row in the cache
        remap.fill_(-7)
        _, misses, _ = L.stem_prefetch_rows_cached(ctx, E_host, torch.from_numpy(ids), E_dev, V, remap, T=T)
        torch.cuda.synchronize()
        assert misses == (0 if batch else distinct.size)
        assert torch.equal(E_dev[remap[:T].long()].cpu(), E_host[torch.from_numpy(ids).long()])
        assert bool((remap[T:] == -7).all())
    ctx.close()
