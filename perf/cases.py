"""The calls of libstem whose speed matters to a program that uses it, over the range of sizes it meets.

Sizes are those of the package's own workloads (`inputs.SHAPES`) or generic ones beside them.  A case is
one of four kinds of pass:

  decode   T single tokens through a stack of layers: one `stem_ffn_forward_residual` call per layer, in
           place on the residual stream.
  prefill  one inference forward of a batch of tokens; with `host` the table lies in pinned host memory and
           the pass is `stem_prefetch_rows` followed by the forward that waits for the rows.
  train    one training step of a layer: forward with saved activations, backward, table gradient and the
           sparse AdamW update of the touched rows, on one stream.
  train_up the same for the layers STEM is compared with: `additive` (up projection plus table) or, without
           it, the dense SwiGLU layer, which has no table and no table update.
"""
import numpy as np
import torch

from paper_2601_10639_amd import inputs, stemlib as L

DEV = "cuda:0"
HP = dict(lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)

BIG = dict(d=2048, F=8192, V=128256)     # the 1B-shaped layer
MID = dict(d=1024, F=4096, V=50304)      # the 350M-shaped layer


def listed():
    return [
        # one user's chat: a single token a step, every weight read once
        dict(name="decode_1", kind="decode", T=1, layers=16, **BIG),
        # a small serving batch on the small model
        dict(name="decode_24_350m", kind="decode", T=24, layers=16, **MID),
        # the decode workload: a full serving batch
        dict(name="decode_256", kind="decode", T=256, layers=16, **BIG),
        # one prompt of a chat, of a length that fits no tile
        dict(name="prefill_700", kind="prefill", T=700, host=False, **BIG),
        # a long document with the table offloaded to host memory
        dict(name="prefill_host_65536", kind="prefill", T=65536, host=True, **BIG),
        # the tiny fp32 layer: reference runs, where launches are everything
        dict(name="train_f32_tiny", kind="train", dtype="f32", T=128, d=64, F=256, V=1000),
        # an fp32 layer of the size at which numerics are compared in earnest
        dict(name="train_f32_1000", kind="train", dtype="f32", T=1000, d=256, F=1024, V=8000),
        # one micro-batch of fine-tuning on a single ragged sequence
        dict(name="train_1999", kind="train", dtype="bf16", T=1999, **BIG),
        # the pre-training steps of the two model shapes
        dict(name="train_350m", kind="train", dtype="bf16", T=16384, **MID),
        dict(name="train_1b", kind="train", dtype="bf16", T=16384, **BIG),
        # long-context training of the small model: more tokens than the one-workgroup sort takes
        dict(name="train_350m_65536", kind="train", dtype="bf16", T=65536, **MID),
        # the comparison layer with both an up projection and a table
        dict(name="train_additive_4096", kind="train_up", additive=True, T=4096, **MID),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _mult(x, m):
    return max(m, int(round(x / m)) * m)


def draw(rng):
    most = 16384 * 2048 * 8192   # T * d * F of the largest training step
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill_host", "train", "train", "train",
                       "train_f32", "train_up"])
    if kind == "train_f32":
        d = _mult(_log(rng, 64, 512), 4)
        F = _mult(d * rng.uniform(2.5, 4.0), 4)
        return dict(kind="train", dtype="f32", T=int(_log(rng, 64, 2048)), d=d, F=F, V=int(_log(rng, 1000, 32000)))
    d = _mult(_log(rng, 512, 2048), 64)
    F = min(8192, _mult(d * rng.uniform(2.5, 4.0), 64))
    V = int(_log(rng, 8000, 128256))
    size = dict(d=d, F=F, V=V)
    if kind == "decode":
        return dict(kind="decode", T=int(_log(rng, 1, 512)), layers=rng.randint(8, 16), **size)
    if kind == "prefill":
        return dict(kind="prefill", T=int(min(_log(rng, 64, 32768), most / d / F)), host=False, **size)
    if kind == "prefill_host":
        return dict(kind="prefill", T=int(_log(rng, 4096, 65536)), host=True, **size)
    if kind == "train":
        return dict(kind="train", dtype="bf16", T=int(min(_log(rng, 128, 65536), most / d / F)), **size)
    return dict(kind="train_up", additive=rng.random() < 0.5, T=int(min(_log(rng, 128, 32768), most / 2 / d / F)), **size)


def _ids(c, seed):
    return inputs.zipf_ids(c["T"], c["V"], seed=seed)


def _distinct(c):
    """Expected number of distinct ids of a case's Zipf(1.1) batch."""
    w = np.arange(1, c["V"] + 1, dtype=np.float64) ** -1.1
    return float(-np.expm1(c["T"] * np.log1p(-w / w.sum())).sum())


def _empty(*shape, dtype=torch.bfloat16):
    return torch.empty(*shape, dtype=dtype, device=DEV)


def _zeros(*shape, dtype=torch.float32):
    return torch.zeros(*shape, dtype=dtype, device=DEV)


def prepare(case, seed):
    c = case
    T, d, F, V = c["T"], c["d"], c["F"], c["V"]
    bf = torch.bfloat16
    if c["kind"] == "decode":
        n = c["layers"]
        ids = torch.from_numpy(_ids(c, seed)).to(DEV)
        k = seed * 1000
        return dict(c=c, ctx=L.stem_create(d, F, V, L.STEM_BF16, T, 0), ids=ids, x=inputs.normal((T, d), 1.0, k, bf, DEV),
                    Wg=[inputs.normal((F, d), 0.02, k + 3 * l + 1, bf, DEV) for l in range(n)],
                    Wd=[inputs.normal((d, F), 0.02, k + 3 * l + 2, bf, DEV) for l in range(n)],
                    E=[inputs.normal((V, F), 0.02, k + 3 * l + 3, bf, DEV) for l in range(n)], y=_empty(T, d))
    if c["kind"] == "prefill":
        s = dict(c=c, ctx=L.stem_create(d, F, V, L.STEM_BF16, T, 0), y=_empty(T, d))
        ids = _ids(c, seed)
        k = seed * 1000
        s["x"] = inputs.normal((T, d), 1.0, k, bf, DEV)
        s["Wg"] = inputs.normal((F, d), 0.02, k + 1, bf, DEV)
        s["Wd"] = inputs.normal((d, F), 0.02, k + 2, bf, DEV)
        E = inputs.normal((V, F), 0.02, k + 3, bf, DEV)
        if c["host"]:
            s["E_host"] = torch.empty(V, F, dtype=bf, pin_memory=True)
            s["E_host"].copy_(E)
            s["ids_host"] = torch.from_numpy(ids)
            s["E_compact"] = _zeros(min(T, V), F, dtype=bf)   # only the first n rows are written
            s["remap"] = _empty(T, dtype=torch.int32)
        else:
            s["E"] = E
            s["ids"] = torch.from_numpy(ids).to(DEV)
        return s

    f32 = c.get("dtype") == "f32"
    dt = torch.float32 if f32 else bf
    up = c["kind"] == "train_up"
    table = not up or c["additive"]
    s = inputs.layer_inputs(inputs.StemShape("case", d, F, V if table else 64, 1, T, "f32" if f32 else "bf16"), seed,
                            device=DEV, ids=_ids(c, seed))
    s.update(c=c, ctx=L.stem_create(d, F, V, L.STEM_F32 if f32 else L.STEM_BF16, T, 0, reserve=L.STEM_RESERVE_UP if up else 0))
    for name, cols in (("y", d), ("G", F), ("H", F), ("dx", d), ("dU", F)):
        s[name] = _empty(T, cols, dtype=dt)
    s["dWg"], s["dWd"] = _empty(F, d, dtype=torch.float32), _empty(d, F, dtype=torch.float32)
    if up:
        s["W_up"] = inputs.normal((F, d), 0.02, seed * 1000 + 7, dt, DEV)
        s["Up"], s["dWu"] = _empty(T, F), _empty(F, d, dtype=torch.float32)
    if table:
        cap = min(T, V)
        s["sorted_ids"], s["perm"] = _empty(T, dtype=torch.int32), _empty(T, dtype=torch.int32)
        # of these only the entries of rows that the batch touches are written
        s["uniq_ids"], s["seg_offsets"] = _zeros(cap, dtype=torch.int32), _zeros(cap + 1, dtype=torch.int32)
        s["n_uniq"] = _zeros(1, dtype=torch.int32)
        s["dE_rows"] = _zeros(cap, F)
        s["master"] = None if f32 else s["E"].float()
        # optimiser state as some way into training: moments of the size of this layer's gradients
        g = 3e-4 if f32 else 0.3
        s["m"] = inputs.normal((V, F), 0.3 * g, seed * 1000 + 8, torch.float32, DEV)
        s["v"] = inputs.normal((V, F), 0.3 * g, seed * 1000 + 9, torch.float32, DEV).abs_().add_(g).square_()
        s["step"] = 1000
    return s


def run(state):
    s = state
    kind = s["c"]["kind"]
    if kind == "decode":
        x = s["x"]
        for Wg, Wd, E in zip(s["Wg"], s["Wd"], s["E"]):
            L.stem_ffn_forward_residual(s["ctx"], x, s["ids"], Wg, Wd, E, x, s["y"])
            x = s["y"]
        return s["y"]
    if kind == "prefill":
        if not s["c"]["host"]:
            L.stem_ffn_forward(s["ctx"], s["x"], s["ids"], s["Wg"], s["Wd"], s["E"], s["y"])
            return s["y"]
        n, ready = L.stem_prefetch_rows(s["ctx"], s["E_host"], s["ids_host"], s["E_compact"], s["remap"])
        L.stem_ffn_forward(s["ctx"], s["x"], s["remap"], s["Wg"], s["Wd"], s["E_compact"], s["y"], wait_event=ready, E_rows=n)
        return {"y": s["y"], "remap": s["remap"], "rows": s["E_compact"], "n": n}

    out = ["y", "dx", "dWg", "dWd", "dU"]
    if kind == "train_up":
        E, ids = (s["E"], s["ids"]) if s["c"]["additive"] else (None, None)
        L.stem_ffn_up_forward(s["ctx"], s["x"], ids, s["W_gate"], s["W_up"], s["W_down"], E, s["y"], s["G"], s["Up"], s["H"])
        L.stem_ffn_up_backward(s["ctx"], s["dy"], s["x"], ids, s["W_gate"], s["W_up"], s["W_down"], E, s["G"], s["Up"],
                               s["H"], s["dx"], s["dWg"], s["dWu"], s["dWd"], s["dU"])
        out.append("dWu")
        if E is None:
            return {k: s[k] for k in out}
    else:
        L.stem_ffn_forward(s["ctx"], s["x"], s["ids"], s["W_gate"], s["W_down"], s["E"], s["y"], s["G"], s["H"])
        L.stem_ffn_backward(s["ctx"], s["dy"], s["x"], s["ids"], s["W_gate"], s["W_down"], s["E"], s["G"], s["H"],
                            s["dx"], s["dWg"], s["dWd"], s["dU"])
    L.stem_embed_grad(s["ctx"], s["ids"], s["dU"], s["sorted_ids"], s["perm"], s["uniq_ids"], s["seg_offsets"],
                      s["n_uniq"], s["dE_rows"])
    L.stem_embed_sparse_adamw(s["ctx"], s["uniq_ids"], s["n_uniq"], s["dE_rows"], s["E"], s["master"], s["m"], s["v"],
                              step=s["step"], **HP)
    s["step"] += 1
    out += ["sorted_ids", "perm", "uniq_ids", "seg_offsets", "n_uniq", "dE_rows", "E", "m", "v"]
    return {k: s[k] for k in out + (["master"] if s["master"] is not None else [])}


def work(case):
    c = case
    T, d, F = c["T"], c["d"], c["F"]
    if c["kind"] == "decode":
        per_layer = 2 * d * F * 2 + _distinct(c) * F * 2
        return {"bytes": c["layers"] * per_layer + 2 * T * d * 2, "flops": c["layers"] * 4 * T * d * F}
    if c["kind"] == "prefill":   # a host-resident table's rows are read over the link and stored once
        rows = _distinct(c) * F * 2
        return {"bytes": 2 * T * d * 2 + 2 * d * F * 2 + rows * (2 if c["host"] else 1), "flops": 4 * T * d * F}
    es = 4 if c.get("dtype") == "f32" else 2
    up = c["kind"] == "train_up"
    mats = 3 if up else 2
    nbytes = 4 * T * d * es + mats * d * F * (es + 4) + T * F * es   # x, dy, y, dx; weights and their gradients; dU
    if not up or c["additive"]:
        # a touched row: read by the forward pass, gradient row, master and two moments read and written
        nbytes += _distinct(c) * F * ((2 * es if es == 2 else 0) + 4 + 24) + 4 * T * 4
    return {"bytes": nbytes, "flops": mats * 6 * T * d * F}


def tolerance(case):
    # About four times the largest distance of any output from the same pass in 64-bit arithmetic:
    #   fp32   rel 6.5e-7, max 8.5e-6 at 1000 tokens (sums up to twice as long are drawn)
    #   decode rel 7.0e-3, max 3.9e-2: sixteen layers, each rounding G, H and the residual stream to bf16
    #   bf16   rel 3.0e-3; max 1.4e-2, and 0.15 where the gradients of one table row cancel
    if case.get("dtype") == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    if case["kind"] == "decode":
        return {"rel": 2.5e-2, "max": 0.16}
    if case["kind"] == "prefill":
        return {"rel": 1e-2, "max": 6e-2}
    return {"rel": 1e-2, "max": 0.6}
