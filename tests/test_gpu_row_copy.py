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
