"""The work that this library does in a 2:4-sparse training run, as cases that can be timed.

Five kinds of case, over the sizes of the workloads in s24_inputs.py and the widths of the gated-activation table in
bench.py, and generic sizes between them:

  step     one training step of one FFN layer through SparseFFN.step: prune and compress (with the mask search, or
           re-applying the stored mask, which is what 39 of 40 steps do), forward, backward, weight gradients with the
           masked decay; bf16, binary16 or fp32, ReLU / GELU / SwiGLU / GEGLU with biases, and the fully sparse mode
           (unbiasedly pruned output gradient)
  forward  SparseFFN.forward alone on few tokens: evaluating or sampling from a layer with sparse weights
  mask     a mask update over the FFN weights of several layers with its monitors: search, flip count, L1-norm gap
  dense    the same layer trained densely, as in the last part of a run: dense GEMMs and weight gradients
  glu      the stand-alone gated activation, forward and backward, on operands in either layout

Weights, activations and output gradients are normal with the standard deviations of s24_inputs.py.
"""
import math

import torch

import paper_2404_01847_amd as s24
from paper_2404_01847_amd.ffn import SparseFFN

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
LAMBDA = 2e-4
LARGEST = 8192 * 8192 * 28672   # tokens x d_model x d_ff of the largest listed step


def _step(name, p, d, f, act, dtype, search=True, mvue=False, bias=False):
    return {"name": name, "kind": "step", "p": p, "d": d, "f": f, "act": act, "dtype": dtype, "search": search,
            "mvue": mvue, "bias": bias}


def listed():
    return [
        # the benchmark's headline layer (workload c5): the widest gated layer, masks searched every step
        _step("step_widest_swiglu", 8192, 8192, 28672, "swiglu", "bf16"),
        # the gated layer as the paper writes it (biases, GELU gate, binary16) at workload c4's size, between two mask
        # updates: the stored mask is re-applied to the updated weights
        _step("step_wide_geglu_f16", 16384, 4096, 11008, "geglu", "f16", search=False, bias=True),
        # workload c3: a GPT-2-large-shaped layer
        _step("step_large_gelu", 16384, 1280, 5120, "gelu", "bf16"),
        # workload c2: a GPT-2-small-shaped layer
        _step("step_small_gelu", 8192, 768, 3072, "gelu", "bf16"),
        # workload c1: the fp32 layer
        _step("step_f32_relu", 512, 256, 1024, "relu", "f32"),
        # one short micro-batch of a GPT-2-small-shaped layer between mask updates: launches and latency
        _step("step_micro_batch", 256, 768, 3072, "gelu", "bf16", search=False),
        # a ragged token count (packed sequences) on a middle-sized gated layer, between mask updates
        _step("step_ragged_swiglu", 3001, 2048, 5504, "swiglu", "bf16", search=False),
        # the fully sparse mode (pruned output gradient, three sparse GEMMs per weight) on a width that is no power of two
        _step("step_mvue_gelu", 4160, 1600, 6400, "gelu", "bf16", mvue=True),
        # sampling: a batch of 16 sequences, one token each, through workload c4's layer
        {"name": "forward_few_tokens", "kind": "forward", "p": 16, "d": 4096, "f": 11008, "act": "swiglu", "dtype": "bf16"},
        # a monitored mask update of six layers of workload c3's model: 12 weights
        {"name": "mask_update_monitored", "kind": "mask", "count": 12, "r": 5120, "q": 1280, "dtype": "bf16", "gap": True},
        # dense fine-tuning step of a layer of width 1024, the last sixth of a run
        {"name": "dense_step", "kind": "dense", "p": 8192, "d": 1024, "f": 4096, "act": "gelu", "dtype": "bf16"},
        # the paper's gated-activation table: 32 x 512 tokens, column-major binary16 input, here with a row-major result
        {"name": "glu_col_to_row", "kind": "glu", "p": 16384, "f": 800, "gate": "geglu", "dtype": "f16", "z_col": True, "h_col": False},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _widths(rng, lo, hi):
    """(d_model, d_ff), multiples of 64, d_ff about 2.5 to 4 times d_model."""
    d = max(1, _log_uniform(rng, lo, hi) // 64)
    f = max(1, int(round(d * rng.choice([2.6875, 3.5, 4.0, rng.uniform(2.5, 4.0)]))))
    return 64 * d, 64 * f


def _tokens(rng, lo, hi):
    p = _log_uniform(rng, lo, hi)
    return p if rng.random() < 0.5 else max(1, p // 64) * 64   # packed sequences, or whole blocks


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["step_f32", "forward", "mask", "dense", "glu"])
    half = rng.choice(["bf16", "bf16", "bf16", "f16"])
    if kind == "step":
        d, f = _widths(rng, 256, 8192)
        p = _tokens(rng, 128, min(16384, LARGEST // (d * f)))
        act = rng.choice(["relu", "gelu", "gelu", "swiglu", "swiglu", "geglu"])
        mvue = rng.random() < 0.25
        c = _step("", max(64, p // 64 * 64) if mvue else p, d, f, act, half, search=rng.random() < 0.4, mvue=mvue,
                  bias=act == "geglu" or rng.random() < 0.25)
    elif kind == "step_f32":
        d, f = _widths(rng, 128, 768)
        c = _step("", _tokens(rng, 64, 1024), d, f, rng.choice(["relu", "gelu", "swiglu"]), "f32", search=rng.random() < 0.5)
    elif kind == "forward":
        d, f = _widths(rng, 768, 8192)
        c = {"kind": "forward", "p": _log_uniform(rng, 1, 256), "d": d, "f": f, "act": rng.choice(["gelu", "swiglu", "swiglu", "geglu"]), "dtype": half}
    elif kind == "mask":
        d, f = _widths(rng, 768, 4096)
        c = {"kind": "mask", "count": rng.choice([1, 2, 6, 12]), "r": f, "q": d, "dtype": rng.choice(["bf16", "bf16", "f16", "f32"]), "gap": rng.random() < 0.5}
    elif kind == "dense":
        d, f = _widths(rng, 512, 4096)
        c = {"kind": "dense", "p": _tokens(rng, 128, 8192), "d": d, "f": f, "act": "gelu", "dtype": half}
    else:
        c = {"kind": "glu", "p": 8 * _log_uniform(rng, 64, 2048), "f": 8 * _log_uniform(rng, 48, 1024), "gate": rng.choice(["swiglu", "geglu"]),
             "dtype": half, "z_col": rng.random() < 0.5, "h_col": rng.random() < 0.5}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------------------------------- inputs
class _Inputs:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, std, dtype):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=dtype) * std


def _layer_weights(rnd, case, dt):
    d, f = case["d"], case["f"]
    up = ("Wg", "Wu") if case["act"] in ("swiglu", "geglu") else ("W1",)
    down = "Wd" if len(up) == 2 else "W2"
    return {**{n: rnd.normal((f, d), 0.02, dt) for n in up}, down: rnd.normal((d, f), 0.02, dt)}


def _make_ffn(rnd, case, dt):
    gated = case["act"] in ("swiglu", "geglu")
    biases = None
    if case.get("bias"):
        names = {"Wgu": 2 * case["f"], "Wd": case["d"]} if gated else {"W1": case["f"], "W2": case["d"]}
        biases = {n: rnd.normal((k,), 0.02, dt) for n, k in names.items()}
    return SparseFFN(_layer_weights(rnd, case, dt), case["p"], case["act"], LAMBDA, concat_gate_up=gated,
                     mvue=case.get("mvue", False), biases=biases)


def prepare(case, seed):
    dt = DTYPES[case["dtype"]]
    rnd = _Inputs(seed)
    s = {"case": case}
    kind = case["kind"]
    if kind in ("step", "forward"):
        s["ffn"] = _make_ffn(rnd, case, dt)
        s["X"] = rnd.normal((case["p"], case["d"]), 1.0, dt)
        if kind == "forward":
            s["ffn"].prune()        # the weights of a layer that is only evaluated are compressed once
        else:
            s["dY"] = rnd.normal((case["p"], case["d"]), 1e-2, dt)
            if not case["search"]:
                s["ffn"].prune()    # the masks of the last update, re-applied by the steps that follow it
    elif kind == "mask":
        r, q, n = case["r"], case["q"], case["count"]
        shapes = [(r, q) if k % 2 == 0 else (q, r) for k in range(n)]
        s["W"] = [rnd.normal(sh, 0.02, dt) for sh in shapes]
        new = lambda shape, t: torch.zeros(shape, dtype=t, device="cuda")
        s["masks"] = [[new((a // 4, b // 4), torch.int16) for _ in range(2)] for a, b in shapes]   # of this and the last update
        for W, (_, old) in zip(s["W"], s["masks"]):
            # the last update's masks: those of slightly different weights
            s24.transposable_mask((W + rnd.normal(tuple(W.shape), 2e-3, dt)).contiguous(), old)
        s["flips"] = [new((1,), torch.int64) for _ in shapes]
        s["gaps"] = [new((a // 4, b // 4), torch.float64) for a, b in shapes] if case["gap"] else None
    elif kind == "dense":
        p, d, f = case["p"], case["d"], case["f"]
        new = lambda *shape: torch.empty(shape, dtype=dt, device="cuda")
        w = _layer_weights(rnd, case, dt)
        s["W1"], s["W2"] = w["W1"], w["W2"]
        # the input-gradient GEMMs read the transposed weights, laid out once per optimizer step
        s["W1T"], s["W2T"] = s["W1"].t().contiguous(), s["W2"].t().contiguous()
        s["X"], s["dY"] = rnd.normal((p, d), 1.0, dt), rnd.normal((p, d), 1e-2, dt)
        s["Z"], s["H"], s["dH"], s["dZ"], s["Y"], s["dX"] = new(p, f), new(p, f), new(p, f), new(p, f), new(p, d), new(p, d)
        s["dW1"] = torch.empty((f, d), dtype=torch.float32, device="cuda")
        s["dW2"] = torch.empty((d, f), dtype=torch.float32, device="cuda")
    else:
        p, f = case["p"], case["f"]
        shape = lambda cols, col_major: (cols, p) if col_major else (p, cols)
        s["Z"] = rnd.normal(shape(2 * f, case["z_col"]), 1.0, dt)
        s["dH"] = rnd.normal(shape(f, case["h_col"]), 1e-2, dt)
        s["H"], s["dZ"] = torch.empty_like(s["dH"]), torch.empty_like(s["Z"])
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        ffn = s["ffn"]
        ffn.step(s["X"], s["dY"], search=case["search"])
        return {"Y": ffn.Y, "dX": ffn.dX, "grads": {n: w.grad for n, w in ffn.w.items()}, "masks": {n: w.mask for n, w in ffn.w.items()},
                "bias_grads": dict(ffn.bias_grad)}
    if kind == "forward":
        return s["ffn"].forward(s["X"])
    if kind == "mask":
        for k, W in enumerate(s["W"]):
            new, old = s["masks"][k]
            s24.transposable_mask(W, new)
            s24.mask_flips(new, old, s["flips"][k])
            if s["gaps"] is not None:
                s24.l1_norm_gap(W, s["gaps"][k])
        return {"masks": [m[0] for m in s["masks"]], "flips": s["flips"], "gaps": s["gaps"]}
    if kind == "dense":
        s24.dense_gemm(s["X"], s["W1"], s["Z"])
        s24.act_fwd(s["Z"], s["H"], s24.ACT_GELU_ERF)
        s24.dense_gemm(s["H"], s["W2"], s["Y"])
        s24.dense_gemm(s["dY"], s["W2T"], s["dH"])
        s24.act_bwd(s["dH"], s["Z"], s["dZ"], s24.ACT_GELU_ERF)
        s24.dense_gemm(s["dZ"], s["W1T"], s["dX"])
        s24.dense_dw_batch([(s["dY"], s["H"], s["dW2"], None, None, 0.0), (s["dZ"], s["X"], s["dW1"], None, None, 0.0)])
        return {"Y": s["Y"], "dX": s["dX"], "dW1": s["dW1"], "dW2": s["dW2"]}
    gate = s24.GATE_SILU if case["gate"] == "swiglu" else s24.GATE_GELU_ERF
    lz, lh = (s24.COL_MAJOR if case[k] else s24.ROW_MAJOR for k in ("z_col", "h_col"))
    s24.glu_fwd(s["Z"], s["H"], gate, layout_z=lz, layout_h=lh)
    s24.glu_bwd(s["dH"], s["Z"], s["dZ"], gate, layout_h=lh, layout_z=lz)
    return {"H": s["H"], "dZ": s["dZ"]}


# ---------------------------------------------------------------------------------------------------- what it takes
def work(case):
    """Inputs read once and outputs written once; of a product with a 2:4 operand only the kept half is counted."""
    es = 4 if case["dtype"] == "f32" else 2
    kind = case["kind"]
    if kind in ("step", "forward", "dense"):
        p, d, f = case["p"], case["d"], case["f"]
        weights = (3 if case["act"] in ("swiglu", "geglu") else 2) * d * f
        product = 2.0 * p * weights            # one pass over all weights, dense
        if kind == "forward":                  # kept values and their positions, X, Y
            return {"bytes": weights * (es / 2 + 1 / 8) + 2 * p * d * es, "flops": product / 2}
        # weights, X and dY in; Y, dX and the fp32 gradients out (and the masks, written by a search, else read)
        masks = weights / 8 if kind == "step" else 0
        sparse = 0 if kind == "dense" else 3 if case["mvue"] else 2
        return {"bytes": weights * (es + 4) + masks + 4 * p * d * es, "flops": product * (3 - sparse / 2)}
    if kind == "mask":                         # weights and old masks in; new masks and, if monitored, gaps out
        cells = case["count"] * case["r"] * case["q"]
        return {"bytes": cells * (es + 2 / 16 + 2 / 16 + (8 / 16 if case["gap"] else 0)), "flops": 0}
    return {"bytes": case["p"] * case["f"] * es * (3 + 5), "flops": 0}


def tolerance(case):
    """About four times the largest difference seen between a case and itself with its sums in another order (blocks of
    64 features and all tokens permuted); for the gated activation, and itself in fp64.  "max" is one unit in the last
    place of the stored type, four times."""
    if case["kind"] == "mask":
        return "exact"       # masks, counts, and gaps of exactly representable sums
    if case["kind"] == "glu":
        return {"rel": 6e-5, "max": {"bf16": 0.032, "f16": 4e-3}[case["dtype"]]}   # measured 1.4e-5 and 6e-6
    if case.get("mvue"):     # a last-bit difference in a gradient can turn a draw: measured 1.1e-4 (bf16), 5.4e-4 (f16)
        return {"rel": 2.2e-3, "max": 0.4}
    if case["dtype"] != "f32" and case["act"] == "relu":   # so can the sign of a sum near zero: measured 4.5e-4
        return {"rel": 2e-3, "max": 0.4}
    # measured at the widest layers: bf16 4.4e-4, f16 1.1e-4, f32 1.2e-6
    return {"bf16": {"rel": 1.8e-3, "max": 0.032}, "f16": {"rel": 5e-4, "max": 5e-3}, "f32": {"rel": 4.8e-6, "max": 3e-5}}[case["dtype"]]
