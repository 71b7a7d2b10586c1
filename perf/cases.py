"""Performance cases of the mixed-batch LoRA linear layer: what a serving and fine-tuning program has this library do.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)` one more of the same ranges.
`prepare(case, seed)` makes what such a program holds before the call (weights, adapters, activations, the context, the
segment table of the batch), `run(state)` is one pass through the public entry points, `work(case)` the bytes and
operations the pass cannot do without, `tolerance(case)` how far two correct implementations may lie apart, `exact(case,
seed)` the outputs in 64 bits.

Three kinds of pass:
  linear    `layers` projections of one shape, each with weights and adapters of its own, on one batch: forward through
            all of them in order and, if the batch trains, backward in reverse order (gradients of every layer).
            micro_batches = 2: a second batch of the same segments adds to the gradients (accumulation).
  siblings  several projections of one input side by side (q, k, v, or gate and up with the SwiGLU epilogue), forward
            and backward; with SwiGLU the backward starts from the gradient of the activated output.
  update    the step after the backward pass: AdamW on the tables of the trained adapters, then the mean of each table
            with the copies of the other replicas.

A batch mixes one-token decode segments, prefill chunks of log-normal length and whole training sequences; adapters
are drawn by a Zipf law (alpha 0: uniform), a share of the inference segments runs on the base weight only.  The batch
is a function of the case (of its "mix"), every tensor a function of the seed.
"""
import math

import numpy as np
import torch

from paper_2604_16400_amd import binding

SCALE = 2.0
MAX_FLOPS = 11.7e12  # one pass of the largest listed case, slightly rounded up


# ----------------------------------------------------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------------------------------------------------
def _linear(name, d_in, d_out, tokens, train, train_segs, decode, adapters, ranks, alpha, base, mix, layers=1, dtype="bf16",
            layout="in_out", micro_batches=1, keep_h=True):
    return {"name": name, "kind": "linear", "d_in": d_in, "d_out": d_out, "tokens": tokens, "train": train,
            "train_segs": train_segs, "decode": decode, "adapters": adapters, "ranks": ranks, "alpha": alpha, "base": base,
            "mix": mix, "layers": layers, "dtype": dtype, "layout": layout, "micro_batches": micro_batches, "keep_h": keep_h}


def _siblings(name, d_in, d_outs, swiglu, tokens, train, train_segs, decode, adapters, ranks, alpha, base, mix):
    return {"name": name, "kind": "siblings", "d_in": d_in, "d_outs": d_outs, "swiglu": swiglu, "tokens": tokens,
            "train": train, "train_segs": train_segs, "decode": decode, "adapters": adapters, "ranks": ranks, "alpha": alpha,
            "base": base, "mix": mix, "dtype": "bf16"}


def listed():
    return [
        # the smallest call of a serving loop: eight requests, one token each, one projection
        _linear("decode_8", 4096, 4096, 8, 0, 0, 8, 16, "16", 0.0, 0.0, 1),
        # a decode step through a stack of MLP projections (each layer's weight comes from memory, the batch stays):
        # adapters of very different ranks and popularity, some requests without one
        _linear("decode_64_layers", 4096, 11008, 64, 0, 0, 64, 64, "8,16,32,128", 1.1, 0.1, 2, layers=4),
        # inference only, ragged: decode tokens beside prefill chunks, odd number of tokens
        _linear("prefill_1003", 5120, 5120, 1003, 0, 0, 200, 32, "32", 1.2, 0.0, 3),
        # a small training step through a stack of attention projections (256 decode tokens + one 1792-token sequence)
        _linear("train_2048_layers", 4096, 4096, 2048, 1792, 1, 256, 16, "16", 0.0, 0.0, 4, layers=4),
        # module-weight layout, h recomputed in the backward pass, gradients accumulated over two micro-batches; sizes
        # that are no multiples of the tiles, ranks that are no multiples of 16
        _linear("accumulate_out_in", 11008, 4104, 1367, 901, 3, 100, 24, "12,20,64", 1.1, 0.05, 5, layout="out_in",
                micro_batches=2, keep_h=False),
        # the ordinary mixed batch with adapters of many ranks: MLP projection, 8192 tokens
        _linear("train_8192_ranks", 5120, 13824, 8192, 3277, 4, 200, 64, "8,16,32,128", 1.1, 0.0, 6),
        # narrow output (grouped-query k or v) over a large batch of 128 rank-16 adapters
        _linear("train_16384_narrow", 8192, 1024, 16384, 8192, 4, 1024, 128, "16", 0.0, 0.0, 7),
        # the largest: MLP projection of a 70B-class model over 16384 tokens
        _linear("train_16384_wide", 8192, 28672, 16384, 8192, 4, 1024, 128, "16", 0.0, 0.0, 8),
        # gate and up in one call with the SwiGLU epilogue, rank 64, 32 adapters of very different popularity
        _siblings("swiglu_4096", 4096, "11008,11008", True, 4096, 1024, 2, 256, 32, "64", 1.2, 0.0, 9),
        # q, k and v in one call over the large batch
        _siblings("qkv_16384", 8192, "8192,1024,1024", False, 16384, 8192, 4, 1024, 128, "16", 0.0, 0.0, 10),
        # fp32: the exact path on a small layer
        _linear("fp32_64", 256, 256, 64, 32, 1, 0, 4, "8", 0.0, 0.0, 11, dtype="f32"),
        # optimizer step and aggregation of the four trained adapters of a large projection
        {"name": "adapter_update", "kind": "update", "d_in": 8192, "d_out": 28672, "rank": 16, "trained": 4, "copies": 4,
         "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, step):
    """A width between lo and hi, over its logarithm: half of them multiples of 256, the others of `step`."""
    q = 256 if lo >= 256 and rng.random() < 0.5 else step
    return max(lo, _log_int(rng, lo, hi) // q * q)


def draw(rng):
    while True:
        case = _draw_once(rng)
        if work(case)["flops"] <= MAX_FLOPS and _addressable(case):
            return case


def _addressable(case):
    """Operand tensors stay below 2 GiB (the layer's limit)."""
    if case["kind"] == "update":
        return True
    e = 2 if case["dtype"] == "bf16" else 4
    d_out = _d_out(case)
    big = max(case["d_in"], d_out)
    return (case["tokens"] + 1) * big * e < 2 ** 31 and (big + 128) * min(case["d_in"], d_out) * e < 2 ** 31


def _draw_once(rng):
    mix = rng.randrange(1 << 30)
    ranks = rng.choice(["8", "16", "32", "64", "128", "8,16,32,128", "12,20,64", "16,64"])
    alpha = rng.choice([0.0, 1.1, 1.2])
    base = rng.choice([0.0, 0.0, 0.1])
    adapters = _log_int(rng, 4, 128)
    kind = rng.choice(["decode", "decode", "prefill", "train", "train", "train", "siblings", "siblings", "fp32", "update"])
    if kind == "decode":
        tokens = _log_int(rng, 1, 256)
        return _strip(_linear("", _width(rng, 1024, 28672, 8), _width(rng, 1024, 28672, 8), tokens, 0, 0, tokens, adapters, ranks,
                              alpha, base, mix, layers=rng.choice([1, 1, 4]), layout=rng.choice(["in_out", "in_out", "out_in"])))
    if kind == "prefill":
        tokens = _log_int(rng, 100, 8192)
        return _strip(_linear("", _width(rng, 1024, 14336, 8), _width(rng, 1024, 14336, 8), tokens, 0, 0, rng.randrange(tokens // 2),
                              adapters, ranks, alpha, base, mix, layout=rng.choice(["in_out", "in_out", "out_in"])))
    if kind == "train":
        tokens = _log_int(rng, 200, 16384)
        train = max(1, int(tokens * rng.uniform(0.2, 0.9)))
        return _strip(_linear("", _width(rng, 1024, 28672, 8), _width(rng, 1024, 28672, 8), tokens, train, rng.randint(1, 4),
                              rng.randrange((tokens - train) // 2 + 1), adapters, ranks, alpha, base, mix,
                              layers=1 if tokens > 2048 else rng.choice([1, 2, 4]), layout=rng.choice(["in_out", "in_out", "out_in"]),
                              micro_batches=1 if tokens > 4096 else rng.choice([1, 1, 2]), keep_h=rng.random() < 0.7))
    if kind == "siblings":
        tokens = _log_int(rng, 200, 16384)
        train = max(1, int(tokens * rng.uniform(0.2, 0.9)))
        swiglu = rng.random() < 0.5
        if swiglu:
            d = _log_int(rng, 1024, 14336) // 256 * 256
            d_outs, r = f"{d},{d}", rng.choice(["16", "32", "64", "16,64"])
        else:
            q = _log_int(rng, 1024, 8192) // 256 * 256
            k = rng.choice([q, max(256, q // 4 // 256 * 256), 1024])
            d_outs, r = f"{q},{k},{k}", rng.choice(["8", "16", "32", "64", "8,16,32"])
        return _strip(_siblings("", _width(rng, 1024, 8192, 8), d_outs, swiglu, tokens, train, rng.randint(1, 4),
                                rng.randrange((tokens - train) // 2 + 1), adapters, r, alpha, base, mix))
    if kind == "fp32":
        tokens = _log_int(rng, 16, 512)
        train = rng.randrange(1, tokens // 2 + 1)
        return _strip(_linear("", _width(rng, 64, 1024, 4), _width(rng, 64, 1024, 4), tokens, train, rng.randint(1, 2),
                              rng.randrange(tokens // 4 + 1), min(adapters, 16), rng.choice(["4", "8", "16", "12,20"]), alpha, base,
                              mix, dtype="f32"))
    return {"kind": "update", "d_in": _width(rng, 1024, 28672, 8), "d_out": _width(rng, 1024, 28672, 8),
            "rank": rng.choice([8, 12, 16, 32, 64, 128]), "trained": rng.randint(1, 4), "copies": rng.randint(2, 8),
            "dtype": rng.choice(["bf16", "bf16", "f32"])}


def _strip(case):
    del case["name"]
    return case


# ----------------------------------------------------------------------------------------------------------------------
# the batch of a case
# ----------------------------------------------------------------------------------------------------------------------
def _d_outs(case):
    return [int(v) for v in case["d_outs"].split(",")] if case["kind"] == "siblings" else [case["d_out"]]


def _d_out(case):
    return sum(_d_outs(case))


def _batch(case):
    """(ranks, seg_start, seg_adapter, seg_is_train) of a case."""
    rng = np.random.Generator(np.random.Philox(key=case["mix"]))
    n = case["adapters"]
    widths = np.array([int(r) for r in case["ranks"].split(",")], dtype=np.int32)
    ranks = rng.choice(widths, size=n).astype(np.int32)
    p = (np.arange(n, dtype=np.float64) + 1.0) ** (-case["alpha"])
    p /= p.sum()
    chunks, left = [], case["tokens"] - case["train"] - case["decode"]
    while left > 0:
        c = min(left, int(np.clip(np.rint(rng.lognormal(5.0, 1.0)), 16, 1024)))
        chunks.append(c)
        left -= c
    inf = rng.choice(n, size=case["decode"] + len(chunks), p=p)
    inf = np.where(rng.random(len(inf)) < case["base"], -1, inf)
    n_tr = min(case["train_segs"], case["train"])
    cuts = [case["train"] * k // max(n_tr, 1) for k in range(n_tr + 1)]
    tr = [cuts[k + 1] - cuts[k] for k in range(n_tr)]
    tr_ad = rng.choice(n, size=n_tr, replace=False, p=p) if n_tr else np.zeros(0, dtype=np.int64)
    lens = np.array([1] * case["decode"] + chunks + tr, dtype=np.int64)
    seg_start = np.zeros(len(lens) + 1, dtype=np.int32)
    seg_start[1:] = np.cumsum(lens)
    seg_adapter = np.concatenate([inf, tr_ad]).astype(np.int32)
    seg_is_train = np.array([0] * (case["decode"] + len(chunks)) + [1] * n_tr, dtype=np.uint8)
    return ranks, seg_start, seg_adapter, seg_is_train


# ----------------------------------------------------------------------------------------------------------------------
# what a program holds before the call
# ----------------------------------------------------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draw:
    """Normal values on the GPU from one seed."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.dtype = dtype

    def __call__(self, shape, std):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=self.dtype).mul_(std)


def prepare(case, seed):
    if case["kind"] == "update":
        return _prepare_update(case, seed)
    rnd = _Draw(seed, _dtype(case))
    ranks, seg_start, seg_adapter, seg_is_train = _batch(case)
    P, d_in, D, T = len(_d_outs(case)), case["d_in"], _d_out(case), case["tokens"]
    flip = case.get("layout") == "out_in"
    shp = (lambda a, b: (b, a)) if flip else (lambda a, b: (a, b))
    max_rank = int(ranks.max()) * P
    trained = set(int(a) for a, t in zip(seg_adapter, seg_is_train) if t)
    small = case["dtype"] == "f32"  # (the small exact layer has small activations)
    std_x, std_a = (0.02, 0.02) if small else (1.0, d_in ** -0.5)
    st = {"case": case, "batch": (ranks, seg_start, seg_adapter, seg_is_train, SCALE), "train": case["train"] > 0,
          "layout": binding.LAYOUT_OUT_IN if flip else binding.LAYOUT_IN_OUT, "d_outs": _d_outs(case),
          "ctx": binding.Context(T, len(seg_adapter), len(ranks), max_rank, max(d_in, D)), "layers": []}
    swiglu = case["kind"] == "siblings" and case["swiglu"]
    f32 = dict(dtype=torch.float32, device="cuda")
    for _ in range(case.get("layers", 1)):
        L = {"W": rnd(shp(d_in, D), 0.02),
             "A": binding.PointerTable([rnd(shp(d_in, int(r) * P), std_a) for r in ranks]),
             "B": binding.PointerTable([rnd(shp(int(r), D), 0.01) for r in ranks]),
             "micro": []}
        for _ in range(case.get("micro_batches", 1)):
            m = {"x": rnd((T, d_in), std_x), "y": torch.zeros((T, D // 2 if swiglu else D), dtype=rnd.dtype, device="cuda")}
            if st["train"]:
                m["h"] = torch.zeros((T, max_rank), **f32) if case.get("keep_h", True) else None
                m["dx"] = torch.zeros((T, d_in), dtype=rnd.dtype, device="cuda")
                if swiglu:
                    m["dout"] = rnd((T, D // 2), 1.0)
                    m["pre"] = torch.zeros((T, D), dtype=rnd.dtype, device="cuda")
                    m["dy"] = torch.zeros((T, D), dtype=rnd.dtype, device="cuda")
                else:
                    m["dy"] = rnd((T, D), 1.0)
            L["micro"].append(m)
        if st["train"]:
            L["dA"] = binding.PointerTable([torch.zeros(shp(d_in, int(r) * P), **f32) if a in trained else None for a, r in enumerate(ranks)])
            L["dB"] = binding.PointerTable([torch.zeros(shp(int(r), D), **f32) if a in trained else None for a, r in enumerate(ranks)])
        st["layers"].append(L)
    return st


def _prepare_update(case, seed):
    rnd = _Draw(seed, torch.float32)
    dt = _dtype(case)
    tables = []
    for _ in range(case["trained"]):
        for shape, std in (((case["d_in"], case["rank"]), case["d_in"] ** -0.5), ((case["rank"], case["d_out"]), 0.01)):
            master = rnd(shape, std)
            t = {"param": master.to(dt), "master": master if case["dtype"] == "bf16" else None, "grad": rnd(shape, 1e-3),
                 "m": rnd(shape, 1e-4), "v": rnd(shape, 1e-3).square_(),
                 "others": [(master + rnd(shape, 0.1 * std)).to(dt) for _ in range(case["copies"] - 1)]}
            t["mean"] = torch.zeros_like(t["param"])
            t["copies"] = binding.PointerTable([t["param"]] + t["others"])
            tables.append(t)
    return {"case": case, "tables": tables}


# ----------------------------------------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------------------------------------
def run(state):
    kind = state["case"]["kind"]
    if kind == "update":
        return _run_update(state)
    return _run_siblings(state) if kind == "siblings" else _run_linear(state)


def _outputs(state):
    out = []
    for L in state["layers"]:
        for m in L["micro"]:
            out += [m[k] for k in ("y", "h", "pre", "dx") if m.get(k) is not None]
            if state["case"]["kind"] == "siblings" and "pre" in m:
                out.append(m["dy"])
        if state["train"]:
            out += [t for t in L["dA"].tensors + L["dB"].tensors if t is not None]
    return out


def _run_linear(state):
    ctx, batch, layout = state["ctx"], state["batch"], state["layout"]
    for k in range(state["case"]["micro_batches"]):
        for L in state["layers"]:
            m = L["micro"][k]
            ctx.collm_lora_linear_fwd(m["x"], L["W"], L["A"], L["B"], *batch, m["y"], m.get("h"), layout=layout)
        if state["train"]:
            for L in reversed(state["layers"]):
                m = L["micro"][k]
                ctx.collm_lora_linear_bwd(m["x"], L["W"], L["A"], L["B"], *batch, m["dy"], m["h"], m["dx"], L["dA"], L["dB"],
                                          accumulate=k > 0, layout=layout)
    return _outputs(state)


def _run_siblings(state):
    ctx, batch, d_outs = state["ctx"], state["batch"], state["d_outs"]
    L = state["layers"][0]
    m = L["micro"][0]
    if state["case"]["swiglu"]:
        ctx.collm_lora_siblings_fwd(d_outs, m["x"], L["W"], L["A"], L["B"], *batch, m["y"], m["h"],
                                    activation=binding.ACT_SWIGLU, pre_act=m["pre"])
        binding.collm_swiglu_bwd(batch[1], batch[3], m["pre"], m["dout"], m["dy"])
    else:
        ctx.collm_lora_siblings_fwd(d_outs, m["x"], L["W"], L["A"], L["B"], *batch, m["y"], m["h"])
    ctx.collm_lora_siblings_bwd(d_outs, m["x"], L["W"], L["A"], L["B"], *batch, m["dy"], m["h"], m["dx"], L["dA"], L["dB"])
    return _outputs(state)


def _run_update(state):
    out = []
    for t in state["tables"]:
        binding.collm_adapter_adamw(t["param"], t["grad"], t["m"], t["v"], 1e-4, 0.9, 0.999, 1e-8, 0.01, 10, master=t["master"])
    for t in state["tables"]:
        binding.collm_adapter_fedavg(t["copies"], t["mean"])
        out += [t["param"], t["m"], t["v"], t["mean"]] + ([t["master"]] if t["master"] is not None else [])
    return out


# ----------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ----------------------------------------------------------------------------------------------------------------------
def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "update":
        n = case["trained"] * case["rank"] * (case["d_in"] + case["d_out"])
        adamw = 4 * 5 + 2 * e if case["dtype"] == "f32" else 4 * 7 + e  # grad, m, v in; m, v out; the weight in and out
        # (the copies of the other replicas in, the mean out; the local copy was just written)
        return {"bytes": n * (adamw + case["copies"] * e), "flops": n * (15 + case["copies"])}
    ranks, seg_start, seg_adapter, seg_is_train = _batch(case)
    lens = np.diff(seg_start).astype(np.int64)
    P, d_in, D, T, Ttr = len(_d_outs(case)), case["d_in"], _d_out(case), case["tokens"], case["train"]
    r_seg = np.where(seg_adapter >= 0, ranks[np.maximum(seg_adapter, 0)], 0).astype(np.int64)
    used = set(int(a) for a, n in zip(seg_adapter, lens) if a >= 0 and n > 0)
    trained = set(int(a) for a, t, n in zip(seg_adapter, seg_is_train, lens) if t and n > 0)
    r_used, r_trained = sum(int(ranks[a]) for a in used), sum(int(ranks[a]) for a in trained)
    swiglu = case["kind"] == "siblings" and case["swiglu"]
    layers, micro = case.get("layers", 1), case.get("micro_batches", 1)
    # low-rank flops per direction: h (d_in, all P tables) and its product with B (D columns)
    low = float((lens * r_seg).sum()) * 2 * (P * d_in + D)
    low_tr = float((lens * r_seg)[seg_is_train != 0].sum()) * 4 * (P * d_in + D)
    flops = 2.0 * (T + Ttr) * d_in * D + low + low_tr
    act = (T * d_in + T * (D // 2 if swiglu else D)) * e              # x in, y out
    if Ttr:
        act += Ttr * d_in * e                                         # dx out
        act += Ttr * (D // 2 + 2 * D if swiglu else D) * e            # dy in (SwiGLU: dout in, pre-activations and dy out)
        if case.get("keep_h", True):
            act += 4 * Ttr * int(ranks.max()) * P                     # h out
    weights = d_in * D * e + r_used * (P * d_in + D) * e              # W and the tables in
    grads = 4 * r_trained * (P * d_in + D)                            # dA and dB out
    return {"bytes": float(layers * (micro * act + weights + grads)), "flops": float(layers * micro * flops)}


def tolerance(case):
    """About four times what the path shows against itself in 64 bits (2-norm / largest element): bf16 1.7e-3 / 1.4e-2,
    with SwiGLU and its gradient in between 3.0e-3 / 2.8e-2, fp32 3e-7 / 1.6e-6 at 256 columns (the sums run over up to 1024)."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    if case["kind"] == "siblings" and case["swiglu"]:
        return {"rel": 1.2e-2, "max": 0.12}
    return {"rel": 7e-3, "max": 0.06}


# ----------------------------------------------------------------------------------------------------------------------
# the same pass in 64 bits
# ----------------------------------------------------------------------------------------------------------------------
def exact(case, seed):
    """What `run` returns for the first pass on these inputs, in fp64 by plain torch: the definition, run of tokens by run of tokens."""
    st = prepare(case, seed)
    return _exact_update(st) if case["kind"] == "update" else _exact_layers(st)


def _exact_layers(st):
    case, (ranks, seg_start, seg_adapter, seg_is_train, scale) = st["case"], st["batch"]
    flip, d_outs = st["layout"] == binding.LAYOUT_OUT_IN, st["d_outs"]
    P, D, swiglu = len(d_outs), sum(d_outs), case["kind"] == "siblings" and case["swiglu"]
    cols = [slice(sum(d_outs[:j]), sum(d_outs[:j + 1])) for j in range(P)]
    wide = lambda t: (t.t() if flip else t).double()
    segs = [(slice(int(seg_start[k]), int(seg_start[k + 1])), int(seg_adapter[k]), bool(seg_is_train[k]))
            for k in range(len(seg_adapter)) if seg_start[k + 1] > seg_start[k]]
    tr = torch.zeros(case["tokens"], dtype=torch.bool, device="cuda")
    for rows, _, t in segs:
        tr[rows] = t
    out = []
    for L in st["layers"]:
        W, A, B = wide(L["W"]), L["A"].tensors, L["B"].tensors
        zeros = lambda table: [torch.zeros_like(wide(t)) if t is not None else None for t in table.tensors]
        dA, dB = (zeros(L["dA"]), zeros(L["dB"])) if st["train"] else ([], [])
        for m in L["micro"]:
            x = m["x"].double()
            y, h = x @ W, torch.zeros((case["tokens"], int(ranks.max()) * P), dtype=torch.float64, device="cuda")
            for rows, a, t in segs:
                if a < 0:
                    continue
                r, hs, b = int(ranks[a]), x[rows] @ wide(A[a]), wide(B[a])
                h[rows, :r * P] = hs
                for j in range(P):
                    y[rows, cols[j]] += scale * (hs[:, j * r:(j + 1) * r] @ b[:, cols[j]])
            pre = y
            if swiglu:
                gate, up = pre[:, :D // 2], pre[:, D // 2:]
                sig = torch.sigmoid(gate)
                y = gate * sig * up
            out.append(y)
            if not st["train"]:
                continue
            zero = lambda t: torch.where(tr[:, None], t, torch.zeros_like(t))
            if m["h"] is not None:
                out.append(zero(h))
            dy = zero(m["dy"].double())
            if swiglu:
                dout = m["dout"].double()
                dy = zero(torch.cat([dout * up * sig * (1 + gate * (1 - sig)), dout * gate * sig], 1))
                out.append(zero(pre))
            dx = zero(dy @ W.t())
            for rows, a, t in segs:
                if not t:
                    continue
                r, hs, b, d = int(ranks[a]), h[rows], wide(B[a]), dy[rows]
                dh = scale * torch.cat([d[:, c] @ b[:, c].t() for c in cols], 1)
                for j in range(P):
                    dB[a][:, cols[j]] += scale * (hs[:, j * r:(j + 1) * r].t() @ d[:, cols[j]])
                dA[a] += x[rows].t() @ dh
                dx[rows] += dh @ wide(A[a]).t()
            out.append(dx)
            if swiglu:
                out.append(dy)
        out += [t.t().contiguous() if flip else t for t in dA + dB if t is not None]
    return out


def _exact_update(st):
    f = lambda v: float(np.float32(v))  # (the hyper-parameters are 32-bit numbers at the boundary)
    lr, b1, b2, eps, wd, step = f(1e-4), f(0.9), f(0.999), f(1e-8), f(0.01), 10
    out = []
    for t in st["tables"]:
        w = (t["master"] if t["master"] is not None else t["param"]).double()
        g = t["grad"].double()
        m = b1 * t["m"].double() + (1 - b1) * g
        v = b2 * t["v"].double() + (1 - b2) * g * g
        w = w * (1 - lr * wd) - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps)
        mean = (w + sum(o.double() for o in t["others"])) / st["case"]["copies"]
        out += [w, m, v, mean] + ([w] if t["master"] is not None else [])
    return out
