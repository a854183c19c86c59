"""Contexts whose host-resident rows cross the link at the same time: what a call on one waits for, and what it leaves to the other."""
import ctypes
import threading

import pytest
import torch

from paper_2601_10639_amd import inputs, stemlib as L
from tests import harness as Hn

DEV = "cuda:0"
NOT_READY = 600   # hipErrorNotReady

pytestmark = pytest.mark.gpu


class LongCopy:
    """A context of 256 KB rows and a call whose rows, 4 GiB, take some 75 ms over the link."""

    def __init__(self):
        T, F = 16384, 65536
        self.E_host = torch.empty(T, F, dtype=torch.float32, pin_memory=True)
        self.E_host[:, 0] = torch.arange(T, dtype=torch.float32)
        self.ids = torch.arange(T, dtype=torch.int32)
        self.E, self.remap = torch.empty(T, F, device=DEV), torch.empty(T, dtype=torch.int32, device=DEV)
        self.ctx = L.stem_create(4, F, T, L.STEM_F32, T, 0)

    def begin(self):
        torch.cuda.synchronize()
        _, self.ready = L.stem_prefetch_rows(self.ctx, self.E_host, self.ids, self.E, self.remap)

    def under_way(self):
        return L.lib().hipEventQuery(ctypes.c_void_p(self.ready)) == NOT_READY

    def end(self):
        torch.cuda.synchronize()
        assert torch.equal(self.E[:, 0].cpu(), self.E_host[:, 0])
        self.E.zero_()


class Layer:
    """A bf16 layer on a host-resident table, checked against the same layer on a device-resident one."""
    T, V, d, F = 500, 3000, 128, 256

    def __init__(self, seed):
        s = inputs.StemShape("beside-a-copy", self.d, self.F, self.V, 1, self.T, "bf16")
        self.inp = inputs.layer_inputs(s, seed=seed, device=DEV, tokens=self.T)
        self.E_host = self.inp["E"].cpu().pin_memory()
        self.E = torch.zeros(2 * self.T, self.F, dtype=torch.bfloat16, device=DEV)
        self.remap = torch.empty(self.T, dtype=torch.int32, device=DEV)
        self.y, self.want = torch.empty_like(self.inp["x"]), torch.empty_like(self.inp["x"])
        self.ctx = Hn.make_ctx(s, self.T)
        L.stem_ffn_forward(self.ctx, self.inp["x"], self.inp["ids"], self.inp["W_gate"], self.inp["W_down"], self.inp["E"], self.want)
        L.stem_sync_status(self.ctx)

    def prefetch(self, ids=None, E=None):
        ids = self.inp["ids"].cpu() if ids is None else ids
        self.n, self.ready = L.stem_prefetch_rows(self.ctx, self.E_host, ids, self.E if E is None else E, self.remap)

    def check(self):
        L.stem_ffn_forward(self.ctx, self.inp["x"], self.remap, self.inp["W_gate"], self.inp["W_down"], self.E, self.y,
                           wait_event=self.ready, E_rows=self.n)
        L.stem_sync_status(self.ctx)
        assert Hn.max_rel(self.y.float().cpu(), self.want.float().cpu()) <= Hn.TOL["bf16"]


@pytest.fixture(scope="module")
def copy():
    c = LongCopy()
    yield c
    c.ctx.close()


def test_a_context_is_made_while_another_ones_rows_are_under_way(copy):
    copy.begin()
    ctx = L.stem_create(64, 64, 64, L.STEM_BF16, 64, 0)
    assert copy.under_way()
    copy.end()
    ctx.close()


@pytest.mark.parametrize("cached", [False, True])
def test_a_refused_call_leaves_the_next_one_nothing_to_wait_for(copy, cached):
    q = Layer(1)
    bad = q.inp["ids"].cpu()
    bad[-1] = q.V
    if cached:
        L.stem_cache_init(q.ctx, q.T)

    def prefetch(ids, cap):
        if cached:
            return L.stem_prefetch_rows_cached(q.ctx, q.E_host, ids, q.E[:q.T + cap], q.T, q.remap)
        return L.stem_prefetch_rows(q.ctx, q.E_host, ids, q.E[:cap], q.remap)

    copy.begin()
    for ids, cap, status in ((bad, q.T, L.STEM_ERR_ID_RANGE), (q.inp["ids"].cpu(), 3, L.STEM_ERR_WORKSPACE)):
        with pytest.raises(L.StemError) as e:
            prefetch(ids, cap)
        assert e.value.status == status
    prefetch(q.inp["ids"].cpu(), q.T)
    assert copy.under_way()
    copy.end()
    q.ctx.close()


def test_short_calls_beside_a_long_one_and_beside_each_other(copy):
    """Rows of a few MB do not wait for another context's 4 GiB, and the rows of two such calls do not all wait for one another."""
    layers = [Layer(k) for k in range(2, 5)]
    copy.begin()
    for q in layers:
        q.prefetch()
    for q in layers:
        L.lib().hipEventSynchronize(ctypes.c_void_p(q.ready))
    assert copy.under_way()
    copy.end()
    for _ in range(3):   # the long call's are done: both streams in turn
        for q in layers:
            q.E.zero_()
        torch.cuda.synchronize()
        for q in layers:
            q.prefetch()
        for q in layers:
            q.check()
    for q in layers:
        q.ctx.close()


def test_a_context_is_closed_while_another_ones_rows_are_under_way(copy):
    gone, stays = Layer(5), Layer(6)
    copy.begin()
    for q in (gone, stays):
        q.prefetch()
    gone.ctx.close()
    stays.check()
    copy.end()
    copy.begin()
    stays.prefetch()
    stays.check()
    copy.end()
    stays.ctx.close()


def test_the_row_cache_beside_another_ones_rows(copy):
    """Promoted rows are copied behind a call's own: hits, misses and promotions of three batches, each beside a long copy."""
    q = Layer(7)
    L.stem_cache_init(q.ctx, 100)
    for k in range(3):
        copy.begin()
        ids = torch.from_numpy(inputs.zipf_ids(q.T, q.V, seed=70 + k))
        _, _, ready = L.stem_prefetch_rows_cached(q.ctx, q.E_host, ids, q.E, 100, q.remap)
        L.stem_ffn_forward(q.ctx, q.inp["x"], q.remap, q.inp["W_gate"], q.inp["W_down"], q.E, q.y, wait_event=ready)
        torch.cuda.current_stream().synchronize()
        assert copy.under_way()
        copy.end()
        assert torch.equal(q.E[q.remap.long()].cpu(), q.E_host[ids.long()])
        state = L.stem_cache_state(q.ctx, 100).long()
        assert torch.equal(q.E[:100][(state >= 0).to(DEV)].cpu(), q.E_host[state[state >= 0]])
    q.ctx.close()


def test_calls_from_two_threads():
    layers = [Layer(8), Layer(9)]
    wrong = []

    def work(q):
        try:
            s = torch.cuda.Stream()
            for _ in range(20):
                q.prefetch()
                L.stem_ffn_forward(q.ctx, q.inp["x"], q.remap, q.inp["W_gate"], q.inp["W_down"], q.E, q.y, wait_event=q.ready,
                                   E_rows=q.n, stream=s)
                s.synchronize()
                if Hn.max_rel(q.y.float().cpu(), q.want.float().cpu()) > Hn.TOL["bf16"]:
                    wrong.append(q)
        except Exception as e:
            wrong.append(e)

    threads = [threading.Thread(target=work, args=(q,)) for q in layers]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for q in layers:
        q.ctx.close()
