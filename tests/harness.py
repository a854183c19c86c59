"""Shared plumbing of the GPU parity tests: runs the HIP path through the C ABI binding and
the oracle on the same seeded inputs.  No arithmetic of the method lives here."""
from __future__ import annotations

import ctypes

import numpy as np
import torch

from oracle import stem_oracle as O
from paper_2601_10639_amd import inputs, stemlib as L

ADAMW = dict(lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)

# Tolerances (max |gpu - ref| / max |ref| per tensor).  fp32 runs accumulate in fp32 over
# at most a few hundred terms: 1e-5.  bf16 runs round G, H, dG, dU, y, dx to bf16 (relative
# 2^-9 each) on top of fp32 accumulation: 2e-2.
TOL = {"f32": 1e-5, "bf16": 2e-2}


def max_rel(got, ref) -> float:
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if ref.size == 0:
        return 0.0
    den = np.abs(ref).max()
    if den == 0:
        return float(np.abs(got).max())
    return float(np.abs(got - ref).max() / den)


def make_ctx(shape: inputs.StemShape, max_tokens: int, reserve: int = 0) -> L.StemCtx:
    dt = L.STEM_BF16 if shape.dtype == "bf16" else L.STEM_F32
    return L.stem_create(shape.d_model, shape.d_ff, shape.vocab, dt, max_tokens, 0, reserve=reserve)


# Which kernel the library chooses, asked through the functions its launchers ask (not part of stem.h).
DECODE, FEW_ROW, TILES = range(3)
EPI_BF16, EPI_F32, EPI_GATE, EPI_DH = range(4)
SORT_ONE_1024, SORT_ONE_4096, SORT_RUNS_1024, SORT_RUNS_4096, SORT_DIGITS = range(5)


def route_tiles(M, N, K, ops=1, epi=EPI_BF16, ws=64 << 20):
    """(kernel, tile rows, tile columns, K slices) of a bf16 product on the large tiles."""
    r = (ctypes.c_int32 * 4)()
    L.lib().stem_route_tiles(M, N, K, ops, epi, ctypes.c_int64(ws), r)
    return tuple(r)


def route_forward(T, d, F):
    """The same for the gate and the down product of a bf16 forward call."""
    r = (ctypes.c_int32 * 8)()
    L.lib().stem_route_forward(d, F, ctypes.c_int64(T), r)
    return tuple(r[:4]), tuple(r[4:])


def route_weight_grads(T, d, F, n, ws=64 << 20):
    """(one launch, tile rows, tile columns, K slices) of a layer's n weight gradients."""
    r = (ctypes.c_int32 * 4)()
    L.lib().stem_route_weight_grads(d, F, ctypes.c_int64(T), n, ctypes.c_int64(ws), r)
    return tuple(r)


def route_weight_grads_apart(T, d, F, **at):
    """Whether they may share a launch, as the buffers lie that are given by name: byte addresses, None for one not there."""
    names = ("dy", "H", "dx", "W_gate", "W_up", "dV", "dW_gate", "dW_up")
    assert set(at) <= set(names)
    return bool(L.lib().stem_route_weight_grads_apart(d, F, ctypes.c_int64(T), *[ctypes.c_void_p(at.get(k)) for k in names]))


def route_gate_up_together(T, d, F, E_rows, **at):
    """Whether the gate and up product may share a launch, as the buffers lie that are given by name: byte addresses, None for one not there."""
    names = ("W_up", "E", "ids", "G", "Up", "H")
    assert set(at) <= set(names)
    p = {k: ctypes.c_void_p(at.get(k)) for k in names}
    return bool(L.lib().stem_route_gate_up_together(d, F, ctypes.c_int64(T), p["W_up"], p["E"], ctypes.c_int64(E_rows), p["ids"], p["G"],
                                                    p["Up"], p["H"]))


def route_sort(T, V):
    return L.lib().stem_route_sort(ctypes.c_int64(T), V)


def route_sort_ranks(T, V, **at):
    """Whether the kernel that counts ranks sorts a call whose buffers lie at these byte addresses."""
    names = ("ids", "sorted_ids", "perm", "uniq_ids", "seg_offsets", "n_uniq", "seg_of")
    assert set(at) <= set(names)
    return bool(L.lib().stem_route_sort_ranks(ctypes.c_int64(T), V, *[ctypes.c_void_p(at.get(k)) for k in names]))


def route_sort_buckets(T, V, **at):
    """Whether buckets of the vocabulary do."""
    names = ("ids", "sorted_ids", "perm", "uniq_ids", "seg_offsets", "n_uniq", "seg_of")
    assert set(at) <= set(names)
    return bool(L.lib().stem_route_sort_buckets(ctypes.c_int64(T), V, *[ctypes.c_void_p(at.get(k)) for k in names]))


def route_sort_sum(bf16, T, V, F, **at):
    """Whether one launch sorts and sums a call whose buffers lie at these byte addresses (seg_of: the context's)."""
    names = ("ids", "dU", "sorted_ids", "perm", "uniq_ids", "seg_offsets", "n_uniq", "seg_of", "dE_rows")
    assert set(at) <= set(names)
    return bool(L.lib().stem_route_sort_sum(int(bf16), ctypes.c_int64(T), V, F, *[ctypes.c_void_p(at.get(k, 0)) for k in names]))


def kernels(ctx, call):
    """{kernel name: launches} of a call on the context."""
    L.stem_profile_enable(ctx, True)
    L.stem_profile_reset(ctx)
    call()
    seen = {k: n for k, (_, n) in L.stem_profile_read(ctx).items()}
    L.stem_profile_enable(ctx, False)
    return seen


def hip_forward_backward(ctx, inp, save_H=True, want_dx=True, after_forward=None):
    """forward + backward through libstem; returns device tensors.  `after_forward()` runs between the two calls."""
    dev = inp["x"].device
    dt = inp["x"].dtype
    T, d = inp["x"].shape
    F = inp["W_gate"].shape[0]
    y = torch.empty(T, d, dtype=dt, device=dev)
    G = torch.empty(T, F, dtype=dt, device=dev)
    H = torch.empty(T, F, dtype=dt, device=dev) if save_H else None
    L.stem_ffn_forward(ctx, inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], y, G, H)
    if after_forward is not None:
        after_forward()
    dx = torch.empty(T, d, dtype=dt, device=dev) if want_dx else None
    dWg = torch.empty(F, d, dtype=torch.float32, device=dev)
    dWd = torch.empty(d, F, dtype=torch.float32, device=dev)
    dU = torch.empty(T, F, dtype=dt, device=dev)
    L.stem_ffn_backward(ctx, inp["dy"], inp["x"], inp["ids"], inp["W_gate"], inp["W_down"], inp["E"], G, H, dx,
                        dWg, dWd, dU)
    return {"y": y, "G": G, "H": H, "dx": dx, "dW_gate": dWg, "dW_down": dWd, "dU": dU}


def hip_embed_grad(ctx, ids, dU, V, with_rows=True, stream=None):
    dev = ids.device
    T = ids.shape[0]
    cap = max(1, min(T, V))
    out = {
        "sorted_ids": torch.empty(max(T, 1), dtype=torch.int32, device=dev),
        "perm": torch.empty(max(T, 1), dtype=torch.int32, device=dev),
        "uniq_ids": torch.empty(cap, dtype=torch.int32, device=dev),
        "seg_offsets": torch.empty(cap + 1, dtype=torch.int32, device=dev),
        "n_uniq": torch.full((1,), -7, dtype=torch.int32, device=dev),
    }
    F = ctx.d_ff
    out["dE_rows"] = torch.empty(cap, F, dtype=torch.float32, device=dev) if with_rows else None
    L.stem_embed_grad(ctx, ids, dU if with_rows else None, out["sorted_ids"], out["perm"], out["uniq_ids"],
                      out["seg_offsets"], out["n_uniq"], out["dE_rows"], T=T, stream=stream)
    return out


def check_integers(eg, ids_np):
    """Bit-exact comparison of the sort / unique outputs with the oracle's."""
    T = len(ids_np)
    s, p = O.sort_ids(ids_np)
    u, offs = O.unique_segments(s)
    U = int(eg["n_uniq"].item())
    assert U == len(u)
    np.testing.assert_array_equal(eg["sorted_ids"][:T].cpu().numpy(), s)
    np.testing.assert_array_equal(eg["perm"][:T].cpu().numpy(), p)
    np.testing.assert_array_equal(eg["uniq_ids"][:U].cpu().numpy(), u)
    np.testing.assert_array_equal(eg["seg_offsets"][:U + 1].cpu().numpy(), offs)
    return U
