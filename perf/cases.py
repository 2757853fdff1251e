"""Performance cases of the MoE layer: the calls a program makes of this library, over the range of sizes,
element types and options they are made with.

A case names a `call` and the layer's sizes:
  layer     moe_layer_forward (moe_layer_forward_aux when `aux`): inference, and the forward of an evaluation
  stages    moe_gate, moe_slice_dispatch, moe_expert_ffn, moe_combine one after another: a program that needs
            the routing or the expert outputs between the stages
  train     moe_layer_forward_train then moe_layer_backward_saved: a training step that keeps intermediates
  backward  moe_layer_backward: the backward of a step that recomputes them (activation checkpointing)

Inputs have the distributions of `paper_2304_11414_amd.synth`: tokens and output gradients N(0, 1), router
and expert weights N(0, 0.02), an optional Zipf router bias.  Everything is drawn on the GPU.
"""

import math

import numpy as np
import torch

from paper_2304_11414_amd import binding as B

_DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(name, call, T, d, F, E, k, local=None, begin=0, cf=0.0, renorm=False, dt="bf16", out=None, zipf_s=0.0,
          zipf_scale=1.0, aux=False):
    c = dict(call=call, T=T, d=d, F=F, E=E, k=k, local=E if local is None else local, begin=begin, cf=cf,
             renorm=renorm, dt=dt, out=dt if out is None else out, zipf_s=zipf_s, zipf_scale=zipf_scale, aux=aux)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # Token generation: one step of a batch of 16 sequences through a layer with 8 experts, top-2.
        # Every expert's weights are read for a handful of rows: latency and weight streaming.
        _case("decode_16_top2", "layer", 16, 2048, 8192, 8, 2, renorm=True),
        # The float32 path at the size it is used at: checking another implementation against it.
        _case("parity_f32", "layer", 256, 256, 1024, 4, 1, dt="f32"),
        # Token generation on one rank of a tensor-parallel group (8 of 64 experts, float32 partial sum):
        # 128 sequences, so about two rows per local expert and some experts without any.
        _case("decode_128_slice", "layer", 128, 4096, 16384, 64, 1, local=8, out="f32"),
        # A prompt of odd length through a layer whose sizes are multiples of 8 only (h = 1000, 4h = 4000),
        # fp16, an expert count that is not a power of two.
        _case("prefill_odd_f16", "layer", 2999, 1000, 4000, 12, 2, renorm=True, dt="f16"),
        # The dense tensor-parallel FFN shard: one expert, a narrow inner size, float32 partial sum.
        _case("dense_shard", "layer", 8192, 2048, 1024, 1, 1, out="f32"),
        # The GPT-style layer (batch 4 x 2048), top-1, no dropping: the headline workload.
        _case("gpt_top1", "layer", 8192, 2048, 8192, 8, 1),
        # Capacity-limited top-2 over 16 experts with a skewed router, and the balance loss.
        _case("capacity_top2_aux", "layer", 16384, 2048, 8192, 16, 2, cf=1.25, renorm=True, zipf_s=1.1, aux=True),
        # One rank of a tensor-parallel group on a full batch: 8 of 64 experts, weights dominate.
        _case("slice_8of64", "layer", 16384, 4096, 16384, 64, 1, local=8, out="f32"),
        # The largest: wide backbone, top-2, heaviest expert about 45 % of the assignments.
        _case("wide_skewed_top2", "layer", 32768, 5120, 20480, 8, 2, renorm=True, zipf_s=1.5, zipf_scale=1.55),
        # Stage by stage, on a batch of 2 x 2048.
        _case("stages_top2", "stages", 4096, 2048, 8192, 16, 2, renorm=True),
        # A training step of the GPT-style layer in fp16, the precision the paper trains in.
        _case("train_gpt_f16", "train", 8192, 2048, 8192, 8, 1, dt="f16", aux=True),
        # The recomputing backward on one rank of the paper's small setting (h = 1024, 8 of 64 experts).
        _case("backward_slice", "backward", 16384, 1024, 4096, 64, 1, local=8, begin=8),
    ]


# What a drawn case may cost: the largest listed one does 4 * 65536 * 5120 * 20480 flop at the rate of the
# 256 x 256 matrix kernels; the general 16-bit kernel (sizes that are not multiples of 64) and the gradient
# products run at a fraction of that rate, float32 at a few per cent.
_MAX_FLOPS = 2.7e13


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        call = rng.choice(["layer", "layer", "layer", "stages", "train", "backward"])
        dt = rng.choice(["bf16", "bf16", "f16"]) if call in ("train", "backward") else rng.choice(["bf16"] * 5 + ["f16"] * 2 + ["f32"])
        odd = rng.random() < 0.2
        if dt == "f32":
            T, d = _log_int(rng, 16, 2048), _log_int(rng, 8, 128) * 8
        else:
            T = _log_int(rng, 256, 32768) if call in ("train", "backward") else _log_int(rng, 1, 32768)
            d = _log_int(rng, 32, 640) * 8 if odd else _log_int(rng, 4, 80) * 64
        F = rng.choice([4 * d, 4 * d, 4 * d, d // 2 // 8 * 8 or 8])
        if odd and dt != "f32":
            F += 8 * rng.randrange(8)
        E = rng.choice([1, 4, 8, 8, 12, 16, 32, 64, 64])
        k = 1 if E == 1 else rng.choice([1, 1, 2, 2, 4])
        local = E if E < 32 or rng.random() < 0.2 else rng.choice([4, 8, 8, 16])
        begin = rng.randrange(E // local) * local
        c = _case("", call, T, d, F, E, k, local=local, begin=begin, cf=rng.choice([0.0, 0.0, 0.0, 1.0, 1.25]),
                  renorm=k > 1, dt=dt, out=dt if dt == "f32" or rng.random() < 0.7 else "f32",
                  zipf_s=rng.choice([0.0, 0.0, 1.1, 1.5]), aux=call in ("layer", "train") and rng.random() < 0.3)
        fast = dt != "f32" and d % 64 == 0 and F % 64 == 0
        most = _MAX_FLOPS / 200 if dt == "f32" else _MAX_FLOPS / 2 if fast else _MAX_FLOPS / 8
        if local < E and _kept(c)[0] < 8:           # (a rank whose experts get no token at all computes nothing)
            continue
        if local * d * F <= 8.5e8 and work(c)["flops"] <= (most / 2 if call in ("train", "backward") else most):
            return c


def _bias(c):
    if not c["zipf_s"]:
        return None
    return -c["zipf_scale"] * c["zipf_s"] * np.log(np.arange(1, c["E"] + 1, dtype=np.float64))


def _config(c):
    return B.make_config(c["T"], c["d"], c["F"], c["E"], c["k"], c["begin"], c["local"], c["cf"], c["renorm"], c["dt"], c["out"])


def _settle_picks(x, Wg, bias, k, g):
    """Draws tokens again whose picks hang on the last bits of a float32 sum: either pick is right for them, and
    two correct implementations would disagree on whole rows."""
    n = min(k + 1, Wg.shape[0])
    todo = torch.arange(x.shape[0], device="cuda")
    while n > 1 and todo.numel():
        bad = []
        for t in todo.split(8192):
            logits = x[t].double() @ Wg.double().t()
            top = torch.topk(logits if bias is None else logits + bias, n, dim=1).values
            bad.append(t[((top[:, :-1] - top[:, 1:]) < 2e-5).any(dim=1)])
        todo = torch.cat(bad)
        if todo.numel():
            x[todo] = torch.empty((todo.numel(), x.shape[1]), dtype=x.dtype, device="cuda").normal_(generator=g)


def prepare(case, seed):
    c, cfg = case, _config(case)
    B.moe_init()
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    dt, odt = _DTYPES[c["dt"]], _DTYPES[c["out"]]
    T, d, F, E, N, k = c["T"], c["d"], c["F"], c["E"], c["local"], c["k"]

    def normal(*shape, std=1.0, dtype=dt):
        t = torch.empty(shape, dtype=dtype, device="cuda")
        t.normal_(0.0, std, generator=g)
        return t

    def empty(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    s = dict(call=c["call"], cfg=cfg, x=normal(T, d), Wg=normal(E, d, std=0.02), W1=normal(N, F, d, std=0.02),
             W2=normal(N, d, F, std=0.02), bias=None)
    b = _bias(c)
    if b is not None:
        s["bias"] = torch.from_numpy(b.astype(np.float32)).cuda()
    _settle_picks(s["x"], s["Wg"], s["bias"], k, g)
    s["aux"] = (empty(1), empty(E), empty(E, dtype=torch.int32)) if c["aux"] else (None, None, None)
    if c["call"] in ("layer", "train"):
        s["out"] = empty(T, d, dtype=odt)
        s["ws"] = empty(B.moe_workspace_bytes(cfg), dtype=torch.uint8)
    if c["call"] in ("train", "backward"):
        s["d_out"] = normal(T, d, dtype=odt)
        s["grads"] = dict(dx=empty(T, d, dtype=dt), dWg=empty(E, d), dbias=empty(E), dW1=empty(N, F, d), dW2=empty(N, d, F))
        s["bws"] = empty(B.moe_layer_backward_workspace_bytes(cfg), dtype=torch.uint8)
        if c["call"] == "train":
            s["saved"] = empty(B.moe_layer_saved_bytes(cfg), dtype=torch.uint8)
    if c["call"] == "stages":
        rows = B.moe_max_rows(cfg)
        i32 = torch.int32
        s.update(idx=empty(T, k, dtype=i32), gate_w=empty(T, k), counts=empty(N, dtype=i32), offsets=empty(N + 1, dtype=i32),
                 perm=empty(rows, dtype=i32), inv_perm=empty(T, k, dtype=i32), xs=empty(rows, d, dtype=dt),
                 H=empty(rows, F, dtype=dt), ys=empty(rows, d, dtype=dt), out=empty(T, d, dtype=odt),
                 dws=empty(B.moe_dispatch_workspace_bytes(cfg), dtype=torch.uint8),
                 fws=empty(B.moe_ffn_workspace_bytes(cfg), dtype=torch.uint8))
    return s


def run(s):
    call, cfg = s["call"], s["cfg"]
    x, Wg, bias, W1, W2 = s["x"], s["Wg"], s["bias"], s["W1"], s["W2"]
    l_aux, mean_prob, first_counts = s["aux"]
    if call == "layer":
        if l_aux is None:
            B.moe_layer_forward(cfg, x, Wg, bias, W1, W2, s["out"], s["ws"])
            return s["out"]
        B.moe_layer_forward_aux(cfg, x, Wg, bias, W1, W2, s["out"], l_aux, mean_prob, first_counts, s["ws"])
        return {"out": s["out"], "l_aux": l_aux, "mean_prob": mean_prob, "first_counts": first_counts}
    if call == "stages":
        B.moe_gate(cfg, x, Wg, bias, None, None, s["idx"], s["gate_w"])
        B.moe_slice_dispatch(cfg, x, s["idx"], s["counts"], s["offsets"], s["perm"], s["inv_perm"], s["xs"], s["dws"])
        B.moe_expert_ffn(cfg, s["xs"], s["offsets"], W1, W2, s["H"], s["ys"], s["fws"])
        B.moe_combine(cfg, s["ys"], s["inv_perm"], s["gate_w"], s["out"])
        return {"out": s["out"], "expert_idx": s["idx"], "gate_w": s["gate_w"], "counts": s["counts"], "inv_perm": s["inv_perm"]}
    gr = s["grads"]
    if call == "backward":
        B.moe_layer_backward(cfg, x, Wg, bias, W1, W2, s["d_out"], gr["dx"], gr["dWg"], gr["dbias"], gr["dW1"], gr["dW2"], s["bws"])
        return gr
    B.moe_layer_forward_train(cfg, x, Wg, bias, W1, W2, s["out"], l_aux, mean_prob, first_counts, s["saved"], s["ws"])
    B.moe_layer_backward_saved(cfg, x, Wg, W1, W2, s["d_out"], s["saved"], gr["dx"], gr["dWg"], gr["dbias"], gr["dW1"], gr["dW2"], s["bws"])
    r = dict(gr, out=s["out"])
    if l_aux is not None:
        r.update(l_aux=l_aux, mean_prob=mean_prob, first_counts=first_counts)
    return r


def _kept(c):
    """(kept assignments of the local experts, local experts with any), estimated from a sample of tokens with
    logits of the distribution the inputs give."""
    rng = np.random.default_rng(1)
    n = min(max(c["T"], 1), 4096)
    lg = rng.standard_normal((n, c["E"])) * 0.02 * math.sqrt(c["d"])
    b = _bias(c)
    if b is not None:
        lg += b
    top = np.argsort(-lg, axis=1)[:, : c["k"]]
    counts = np.bincount(top.ravel(), minlength=c["E"]) * (c["T"] / n)
    if c["cf"] > 0:
        counts = np.minimum(counts, math.ceil(c["cf"] * c["k"] * c["T"] / c["E"]))
    counts = counts[c["begin"] : c["begin"] + c["local"]]
    return float(counts.sum()), int((counts > 0).sum())


def work(case):
    c = case
    rows, used = _kept(c)
    T, d, F, E, N, k = c["T"], c["d"], c["F"], c["E"], c["local"], c["k"]
    eb, ob = (4 if c["dt"] == "f32" else 2), (4 if c["out"] == "f32" else 2)
    gemm = 2.0 * rows * d * F                      # one product of the expert FFN
    router = 2.0 * T * d * E
    weights = 2.0 * used * d * F * eb
    fwd = T * d * eb + E * d * eb + weights + T * d * ob
    if c["call"] == "layer":
        return {"bytes": fwd, "flops": 2 * gemm + router}
    if c["call"] == "stages":                      # the stages' own results: sliced tokens, H, expert outputs
        return {"bytes": fwd + 2 * rows * (2 * d + F) * eb, "flops": 2 * gemm + router}
    grads = T * d * eb + E * d * 4 + 2.0 * N * d * F * 4
    bwd = T * d * (eb + ob) + E * d * eb + weights + grads
    if c["call"] == "backward":                    # the first product again, and four gradient products
        return {"bytes": bwd, "flops": 5 * gemm + 3 * router}
    kept = rows * (d + 2 * F) * eb                 # sliced tokens and both sides of the activation: written, then read
    return {"bytes": fwd + bwd + 2 * kept, "flops": 6 * gemm + 3 * router}


def tolerance(case):
    """Four times what the outputs were measured to be off an evaluation in float64 with the same picks.  Layer
    outputs: 2.9e-3 in bf16, 3.6e-4 in fp16, 1.9e-6 in float32.  A training step's: 5.2e-3 and 1.0e-3 (the bias
    gradient, a column sum with cancellation; the other gradients 3.8e-3 and 4.7e-4).  The largest element
    is off by 3.4e-2, 4.1e-3, 1.7e-5 of the root mean square, which rows without a local expert (zeros) dilute."""
    rel, most = {"bf16": (1.2e-2, 0.14), "f16": (1.5e-3, 0.017), "f32": (8e-6, 7e-5)}[case["dt"]]
    if case["call"] in ("train", "backward"):
        rel = {"bf16": 2.1e-2, "f16": 4e-3}[case["dt"]]
    return {"rel": rel, "max": min(0.9, most * math.sqrt(case["E"] / case["local"]))}
