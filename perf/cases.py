"""Performance cases of the library's main paths, through the Python binding.

A case is a plain dict; ``prepare`` builds what a program holds before the call (inputs, packed
deltas, scales, output buffers of the serving paths, plans of the batched entry points) and ``run``
is one call.  Five kinds of work:

  linear    Y = X W_hat^T of one layer: decode (1-64 tokens) and prefill (more), per-row,
            per-column or blockwise scales
  stack     decode of several transformer blocks' layers through the batched entry point
  variants  requests of different fine-tunes that share one base layer
  grad      gradient with respect to the scale vector (fitting the scales)
  pack      compression of a block's layers, or of one layer, from a base / fine-tuned pair
  patch     merging a block's deltas, or one layer's, into the weights
"""
import math

import torch

from paper_2512_19720_amd import binding as pd
from paper_2512_19720_amd import synth

DEV = "cuda:0"
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
AXES = {"row": pd.ROW, "col": pd.COL}
DECODE_MAX_TOKENS = 64


def listed():
    return [
        # the smallest layer of the test configurations: launch and host latency
        {"name": "linear_small", "kind": "linear", "M": 4, "d_out": 256, "d_in": 512, "dtype": "f16", "scales": "row"},
        # single-stream decode of an attention projection
        {"name": "decode_1", "kind": "linear", "M": 1, "d_out": 4096, "d_in": 4096, "dtype": "f16", "scales": "row"},
        # decode of a batch of 16 sequences, down projection, column scales
        {"name": "decode_16", "kind": "linear", "M": 16, "d_out": 4096, "d_in": 11008, "dtype": "bf16", "scales": "col"},
        # a ragged batch near the end of the decode range on a gate / up projection
        {"name": "decode_61", "kind": "linear", "M": 61, "d_out": 11008, "d_in": 4096, "dtype": "bf16", "scales": "row"},
        # decode of independent layers in one launch: the 14 projections of two blocks, one with
        # row and one with column scales
        {"name": "decode_stack", "kind": "stack", "M": 1, "layers": 14, "dtype": "f16"},
        # sixteen requests for sixteen fine-tunes of one base
        {"name": "variants_16", "kind": "variants", "R": 16, "d_out": 4096, "d_in": 4096, "dtype": "f16", "scales": "row"},
        # a short prompt of odd length
        {"name": "prefill_251", "kind": "linear", "M": 251, "d_out": 4096, "d_in": 4096, "dtype": "f16", "scales": "col"},
        # blockwise scales on a medium prompt
        {"name": "prefill_777_group", "kind": "linear", "M": 777, "d_out": 4096, "d_in": 11008, "dtype": "bf16", "scales": "g128"},
        # a long prompt: the benchmark's prefill shape
        {"name": "prefill_2048", "kind": "linear", "M": 2048, "d_out": 11008, "d_in": 4096, "dtype": "bf16", "scales": "row"},
        # one backward step of fitting the scales on 2048 calibration tokens
        {"name": "grad_2048", "kind": "grad", "M": 2048, "d_out": 4096, "d_in": 4096, "dtype": "bf16", "scales": "col"},
        # compression of one block: seven layers, signs and both scale vectors
        {"name": "pack_block", "kind": "pack", "layers": 7, "d_out": 0, "d_in": 0, "dtype": "f16", "scales": "both"},
        # hot-swap merge of one block's deltas
        {"name": "patch_block", "kind": "patch", "layers": 7, "d_out": 0, "d_in": 0, "dtype": "bf16", "scales": "row"},
    ]


# the most arithmetic that one call of the listed cases does
MAX_FLOPS = 2 * 2048 * 11008 * 4096
# the weights of one block
BLOCK_WEIGHTS = sum(d_out * d_in for _, d_out, d_in in synth.STACK_BLOCK)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _features(rng, lo, hi, step):
    return max(step, int(round(_log(rng, lo, hi) / step)) * step)


def draw(rng):
    """One more case.  Layer shapes spread over 256 to 14336 outputs and 512 to 11008 inputs; the
    outputs are any whole number now and then, the inputs mostly a multiple of 128 and always of 32
    (the packing's own rule)."""
    kind = rng.choice(("decode", "decode", "decode", "prefill", "prefill", "prefill", "stack", "variants", "grad", "pack", "patch"))
    dtype = rng.choice(("f16", "bf16"))
    d_out = rng.randint(256, 4096) if rng.random() < 0.25 else _features(rng, 256, 14336, 64)
    d_in = _features(rng, 512, 11008, 32 if rng.random() < 0.25 else 128)
    if kind in ("decode", "prefill"):
        M = max(1, int(_log(rng, 1, 65))) if kind == "decode" else int(_log(rng, 65, 2049))
        M = min(M, MAX_FLOPS // (2 * d_out * d_in))
        scales = rng.choice(("row", "row", "col", "col", "group"))
        if scales == "group":
            fits = [g for g in (32, 64, 128) if d_in % g == 0]
            scales = rng.choice(["scalar"] + ["g%d" % g for g in fits])
        return {"kind": "linear", "M": M, "d_out": d_out, "d_in": d_in, "dtype": dtype, "scales": scales}
    if kind == "stack":
        return {"kind": "stack", "M": rng.choice((1, 1, 1, 2, 3, 4, 6, 8)), "layers": rng.randint(2, 14), "dtype": dtype}
    if kind == "variants":
        return {"kind": "variants", "R": int(_log(rng, 2, 17)), "d_out": d_out, "d_in": max(128, d_in // 128 * 128), "dtype": dtype,
                "scales": rng.choice(("row", "col", "mixed"))}
    if kind == "grad":
        d_out = max(32, d_out // 32 * 32)
        M = min(int(_log(rng, 64, 4097)), MAX_FLOPS // (2 * d_out * d_in))
        return {"kind": "grad", "M": M, "d_out": d_out, "d_in": d_in, "dtype": dtype, "scales": rng.choice(("row", "col"))}
    layers = max(1, min(rng.choice((1, 1, rng.randint(2, 12))), BLOCK_WEIGHTS // (d_out * d_in)))
    if kind == "pack":
        scales = "both" if layers > 1 else rng.choice(("both", "both", "row", "col", "g128" if d_in % 128 == 0 else "both", "scalar"))
    else:
        scales = rng.choice(("row", "col"))
    return {"kind": kind, "layers": layers, "d_out": d_out, "d_in": d_in, "dtype": dtype, "scales": scales}


# ---- inputs -----------------------------------------------------------------------------------

def _seeds(seed):
    g = torch.Generator()
    g.manual_seed(seed)
    while True:
        yield int(torch.randint(1, 2 ** 31 - 1, (1,), generator=g))


def _generator(seeds):
    g = torch.Generator(device=DEV)
    g.manual_seed(next(seeds))
    return g


def _weights(d_out, d_in, dtype, seeds):
    return torch.randn((d_out, d_in), generator=_generator(seeds), device=DEV, dtype=torch.float32).mul_(synth.W_STD).to(DTYPES[dtype])


def _tokens(M, n, dtype, seeds, scale=1.0):
    return torch.randn((M, n), generator=_generator(seeds), device=DEV, dtype=torch.float32).mul_(scale).to(DTYPES[dtype])


def _signs(d_out, d_in, seeds):
    return torch.randint(-2 ** 31, 2 ** 31, (d_out, d_in // 32), generator=_generator(seeds), device=DEV, dtype=torch.int64).to(torch.int32)


def _scales(shape, seeds):
    """Mean |dW| of a Gaussian delta whose standard deviation is log-normal from channel to channel."""
    z = torch.randn(shape, generator=_generator(seeds), device=DEV, dtype=torch.float32)
    return (torch.exp(z * synth.SIGMA_LOG_STD + synth.SIGMA_LOG_MEAN) * math.sqrt(2 / math.pi)).to(torch.float16)


def _delta(d_out, d_in, scales, seeds):
    v_len = d_out if scales == "row" else d_in
    return _signs(d_out, d_in, seeds), _scales(v_len, seeds)


def _group(case):
    """(group, rows of the scale matrix) of a blockwise or scalar case."""
    if case["scales"] == "scalar":
        return case["d_in"], 1
    return int(case["scales"][1:]), case["d_out"]


def _layers(case):
    """(d_out, d_in) of each layer: the block's own, or several of one size."""
    if case["d_out"]:
        return [(case["d_out"], case["d_in"])] * case["layers"]
    return [(d_out, d_in) for _, d_out, d_in in synth.STACK_BLOCK]


def _stack(case):
    """(scales, d_out, d_in) of each layer of a stack: block after block, the first with row scales,
    the next with column scales."""
    per = len(synth.STACK_BLOCK)
    return [(("row", "col")[k // per % 2], *synth.STACK_BLOCK[k % per][1:]) for k in range(case["layers"])]


def prepare(case, seed):
    seeds, dtype, kind = _seeds(seed), case["dtype"], case["kind"]
    st = {"case": case}
    if kind == "linear":
        M, d_out, d_in = case["M"], case["d_out"], case["d_in"]
        st["X"] = _tokens(M, d_in, dtype, seeds)
        st["W_b"] = _weights(d_out, d_in, dtype, seeds)
        if case["scales"] in AXES:
            st["B"], st["v"] = _delta(d_out, d_in, case["scales"], seeds)
        else:
            group, rows = _group(case)
            st["B"], st["v"] = _signs(d_out, d_in, seeds), _scales((rows, d_in // group), seeds)
        # a decode loop writes into the same activation buffer at every step
        st["Y"] = torch.empty((M, d_out), dtype=DTYPES[dtype], device=DEV) if M <= DECODE_MAX_TOKENS else None
    elif kind == "stack":
        items = []
        for scales, d_out, d_in in _stack(case):
            X, W_b = _tokens(case["M"], d_in, dtype, seeds), _weights(d_out, d_in, dtype, seeds)
            items.append((X, W_b, *_delta(d_out, d_in, scales, seeds), AXES[scales]))
        st["plan"] = pd.pdelta_linear_batch_plan(items)
    elif kind == "variants":
        R, d_out, d_in = case["R"], case["d_out"], case["d_in"]
        axes = [("row", "col")[r % 2] if case["scales"] == "mixed" else case["scales"] for r in range(R)]
        st["X"], st["W_b"] = _tokens(R, d_in, dtype, seeds), _weights(d_out, d_in, dtype, seeds)
        deltas = [_delta(d_out, d_in, a, seeds) for a in axes]
        st["variants"] = pd.VariantSet(deltas, [AXES[a] for a in axes] if case["scales"] == "mixed" else AXES[case["scales"]])
        st["Y"] = torch.empty((R, d_out), dtype=DTYPES[dtype], device=DEV)
    elif kind == "grad":
        st["X"] = _tokens(case["M"], case["d_in"], dtype, seeds)
        st["dY"] = _tokens(case["M"], case["d_out"], dtype, seeds, scale=0.1)
        st["B"] = _signs(case["d_out"], case["d_in"], seeds)
    elif kind == "pack":
        pairs = []
        for d_out, d_in in _layers(case):
            L = synth.layer_device(d_out, d_in, synth.BF16 if dtype == "bf16" else synth.F16, "row", next(seeds), DEV, zero_frac=0.05, with_wf=True)
            pairs.append((L["W_f"], L["W_b"]))
        st["pairs"] = pairs
        st["plan"] = pd.pdelta_pack_batch_plan(pairs) if case["layers"] > 1 else None
    elif kind == "patch":
        items = []
        for d_out, d_in in _layers(case):
            W_b = _weights(d_out, d_in, dtype, seeds)
            items.append((W_b, *_delta(d_out, d_in, case["scales"], seeds), AXES[case["scales"]], torch.empty_like(W_b)))
        st["items"] = items
        st["plan"] = pd.pdelta_patch_batch_plan(items) if case["layers"] > 1 else None
    else:
        raise ValueError(kind)
    return st


# ---- one pass ---------------------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind, scales = case["kind"], case["scales"] if "scales" in case else None
    if kind == "linear":
        if scales == "row":
            return pd.pdelta_linear_row(st["X"], st["W_b"], st["B"], st["v"], out=st["Y"])
        if scales == "col":
            return pd.pdelta_linear_col(st["X"], st["W_b"], st["B"], st["v"], out=st["Y"])
        return pd.pdelta_linear_group(st["X"], st["W_b"], st["B"], st["v"], _group(case)[0], out=st["Y"])
    if kind == "stack":
        return pd.pdelta_linear_batch(st["plan"])
    if kind == "variants":
        return pd.pdelta_linear_variants(st["X"], st["W_b"], st["variants"], out=st["Y"])
    if kind == "grad":
        return pd.pdelta_grad_v(st["X"], st["dY"], st["B"], AXES[scales])
    if kind == "pack":
        if st["plan"] is not None:
            return pd.pdelta_pack_batch(st["plan"])
        W_f, W_b = st["pairs"][0]
        if scales in ("both", "row", "col"):
            got = pd.pdelta_pack(W_f, W_b, want_row=scales != "col", want_col=scales != "row")
            return [t for t in got if t is not None]
        return pd.pdelta_pack_group(W_f, W_b, _group(case)[0], shared_rows=scales == "scalar")
    if st["plan"] is not None:
        return pd.pdelta_patch_batch(st["plan"])
    W_b, B, v, axis, W_out = st["items"][0]
    return pd.pdelta_patch(W_b, B, v, axis, out=W_out)


# ---- what a pass cannot do without, and how exact it is -----------------------------------------

def work(case):
    """Bytes: every weight, sign word, scale, activation once in, every result once out."""
    kind = case["kind"]
    if kind in ("linear", "variants"):
        d_out, d_in = case["d_out"], case["d_in"]
        M, sets = (case["M"], 1) if kind == "linear" else (case["R"], case["R"])
        if kind == "linear" and case["scales"] not in AXES:
            group, rows = _group(case)
            v_len = rows * (d_in // group)
        elif case["scales"] == "mixed":
            v_len = (d_out + d_in) // 2
        else:
            v_len = d_out if case["scales"] == "row" else d_in
        return {"bytes": 2 * d_out * d_in + sets * (d_out * d_in // 8 + 2 * v_len) + 2 * M * (d_in + d_out), "flops": 2 * M * d_out * d_in}
    if kind == "stack":
        nbytes = flops = 0
        for scales, d_out, d_in in _stack(case):
            nbytes += 2 * d_out * d_in + d_out * d_in // 8 + 2 * (d_out if scales == "row" else d_in) + 2 * case["M"] * (d_in + d_out)
            flops += 2 * case["M"] * d_out * d_in
        return {"bytes": nbytes, "flops": flops}
    if kind == "grad":
        M, d_out, d_in = case["M"], case["d_out"], case["d_in"]
        return {"bytes": 2 * M * (d_in + d_out) + d_out * d_in // 8 + 4 * (d_out if case["scales"] == "row" else d_in), "flops": 2 * M * d_out * d_in}
    nbytes = flops = 0
    for d_out, d_in in _layers(case):
        n = d_out * d_in
        if kind == "pack":
            v_len = {"both": d_out + d_in, "row": d_out, "col": d_in, "scalar": 1, "g128": n // 128}[case["scales"]]
            nbytes += 4 * n + n // 8 + 2 * v_len
            flops += 2 * n
        else:
            nbytes += 4 * n + n // 8 + 2 * (d_out if case["scales"] == "row" else d_in)
            flops += n
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Packed signs, scales and merged weights are one rounding of an exact value.  The others are
    about four times the distance from a 64-bit evaluation: a linear layer carries the rounding of
    its 16-bit output (fp16: 2.1e-4, bf16: 1.7e-3) and in prefill that of the fp16 weight tile
    (together 2.9e-4 with fp16 outputs); a gradient is a sum in 32 bits (1.4e-7)."""
    kind = case["kind"]
    if kind in ("pack", "patch"):
        return "exact"
    if kind == "grad":
        return {"rel": 1e-6, "max": 5e-6}
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    if kind == "linear" and case["M"] > DECODE_MAX_TOKENS:
        return {"rel": 1.2e-3, "max": 5e-3}
    return {"rel": 8e-4, "max": 2e-3}


# ---- the same results in 64 bits ----------------------------------------------------------------

def _signs64(B, d_in):
    bits = (B.unsqueeze(-1) >> torch.arange(32, dtype=torch.int32, device=B.device)) & 1
    return (bits.reshape(B.shape[0], d_in) * 2 - 1).double()


def _merged64(W_b, B, v, scales, group=0):
    signs, v = _signs64(B, W_b.shape[1]), v.double()
    if scales == "row":
        v = v.unsqueeze(1)
    elif scales != "col":
        v = v.repeat_interleave(group, dim=1)
    return signs.mul_(v).add_(W_b.double())


def exact(case, seed):
    """What run() returns, in 64 bits; the sign words have no such value."""
    st, kind, scales = prepare(case, seed), case["kind"], case.get("scales")
    if kind == "linear":
        group = 0 if scales in AXES else _group(case)[0]
        return st["X"].double() @ _merged64(st["W_b"], st["B"], st["v"], scales, group).T
    if kind == "stack":
        out = []
        for (scales, _, _), (X, W_b, B, v, _) in zip(_stack(case), st["plan"].tensors):
            out.append(X.double() @ _merged64(W_b, B, v, scales).T)
        return out
    if kind == "variants":
        # the same draws as in prepare(), which hands the deltas to the library
        seeds, d_out, d_in = _seeds(seed), case["d_out"], case["d_in"]
        _tokens(1, 1, case["dtype"], seeds), _weights(1, 1, case["dtype"], seeds)
        rows = []
        for r in range(case["R"]):
            axis = ("row", "col")[r % 2] if scales == "mixed" else scales
            rows.append(st["X"][r:r + 1].double() @ _merged64(st["W_b"], *_delta(d_out, d_in, axis, seeds), axis).T)
        return torch.cat(rows)
    if kind == "grad":
        X, dY, signs = st["X"].double(), st["dY"].double(), _signs64(st["B"], case["d_in"])
        return (dY * (X @ signs.T)).sum(0) if scales == "row" else (X * (dY @ signs)).sum(0)
    if kind == "pack":
        out = []
        for W_f, W_b in st["pairs"]:
            size = (W_f.double() - W_b.double()).abs_()
            if scales in ("both", "row", "col"):
                means = [size.mean(1) if scales != "col" else None, size.mean(0) if scales != "row" else None]
                out.append([None] + [m for m in means if m is not None])
            elif scales == "scalar":
                out.append([None, size.mean().reshape(1, 1)])
            else:
                out.append([None, size.reshape(size.shape[0], -1, _group(case)[0]).mean(2)])
        return out if st["plan"] is not None else out[0]
    out = [_merged64(W_b, B, v, scales) for W_b, B, v, _, _ in st["items"]]
    return out if st["plan"] is not None else out[0]
