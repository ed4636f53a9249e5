"""Performance cases: the work that users of this package have it do, through its public entry points.

Four kinds of work, each over the sizes the package's workloads, tests and benchmark use:

  train      one rank's share of a training iteration of a pipeline stage: the gradient accumulators are cleared,
             then the braid steps of the stage's schedule (F, F&B, F&W, F&BW, BW, B, W blocks) run for every
             microbatch, on three streams or, `serial`, on one; bf16 layers of all kinds and the fp32 configuration
  forward    the F units of consecutive layers called one by one on the current stream (evaluation, prefill)
  attention  the attention core alone, forward then backward (long contexts, many short sequences)
  rows       the memory-bound row and elementwise kernels alone, forward and backward

A case is a dict of plain values; `prepare` builds on the GPU what such a program holds (weights, activations,
stashes, the context with its workspace, the op lists), `run` is one pass."""
from __future__ import annotations

import ctypes as C
import math

import torch

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import binding as B
from paper_2510_27257_amd import stage as S
from paper_2510_27257_amd.synth import Workload

_GPT = dict(norm="ln", act="gelu", causal=True, rope=False, has_bias=True)
_LLAMA = dict(norm="rms", act="swiglu", causal=True, rope=True, has_bias=False)


def _layer(hidden, heads, kv_heads, head_dim, ffn, seq, mbsz, tp, dtype="bf16", **options):
    return dict(hidden=hidden, heads=heads, kv_heads=kv_heads, head_dim=head_dim, ffn=ffn, seq=seq, mbsz=mbsz, tp=tp, dtype=dtype, **options)


def listed():
    return [
        # the smallest configuration, an unsharded fp32 layer of hidden 256 over 128 tokens: launches and latency count
        dict(name="tiny_fp32", kind="train", layers=1, microbatches=2, serial=False, **_layer(256, 4, 4, 64, 1024, 128, 1, 1, dtype="f32", **_GPT)),
        # the headline layer (GPT-7B shape, TP=8 shard, 6144 tokens): forward passes braided with full backward passes
        dict(name="gpt7b_tp8", kind="train", layers=1, microbatches=3, serial=False, **_layer(4096, 4, 4, 128, 2048, 6144, 1, 8, **_GPT)),
        # Llama-13B shape, TP=4 shard (SwiGLU, RMSNorm, RoPE), the steps in order on one stream
        dict(name="llama13b_tp4_serial", kind="train", layers=1, microbatches=2, serial=True, **_layer(5120, 10, 10, 128, 3456, 4096, 1, 4, **_LLAMA)),
        # grouped-query attention, 5 query heads on one key / value head, FFN shard of 1728 columns
        dict(name="gqa12b_tp8_s3072", kind="train", layers=1, microbatches=3, serial=False, **_layer(5120, 5, 1, 128, 1728, 3072, 1, 8, **_LLAMA)),
        # the widest shard of the model table: hidden 7168, 14 query heads on 2 key / value heads, FFN shard of 5120
        dict(name="gqa26b_tp4", kind="train", layers=1, microbatches=2, serial=False, **_layer(7168, 14, 2, 128, 5120, 4096, 1, 4, **_LLAMA)),
        # the vision-encoder layers of a multimodal stage: bidirectional, head dimension 64, 1024 tokens
        dict(name="vit_x2", kind="train", layers=2, microbatches=4, serial=False, **_layer(1024, 16, 16, 64, 4096, 1024, 1, 1, **dict(_GPT, causal=False))),
        # a four-layer pipeline stage over eight microbatches, every block kind of the schedule: the largest job
        dict(name="stage_4x8", kind="train", layers=4, microbatches=8, serial=False, **_layer(4096, 4, 4, 128, 2048, 4096, 1, 8, **_GPT)),
        # nothing a power of two: hidden 1032, FFN 2744, three sequences of 1000 tokens, 6 heads on 2 of dimension 64
        dict(name="ragged", kind="train", layers=1, microbatches=2, serial=True, **_layer(1032, 6, 2, 64, 2744, 1000, 3, 4, **_LLAMA)),
        # evaluation: forward passes only, two layers with grouped-query attention over 6144 tokens
        dict(name="forward_gqa12b_tp4", kind="forward", layers=2, **_layer(5120, 10, 2, 128, 3456, 6144, 1, 4, **_LLAMA)),
        # long context: one causal sequence of 16384 tokens, attention forward and backward
        dict(name="attention_16k", kind="attention", heads=4, kv_heads=4, head_dim=128, seq=16384, mbsz=1, causal=True),
        # many short sequences in one microbatch
        dict(name="attention_short", kind="attention", heads=8, kv_heads=8, head_dim=64, seq=520, mbsz=8, causal=True),
        # the memory-bound kernels at the headline layer's activation size
        dict(name="rows_6144x4096", kind="rows", rows=6144, width=4096),
    ]


def _log_int(rng, lo, hi, step):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _heads(rng, most):
    kv = rng.choice([1, 1, 2, 3, 4, 8])
    group = rng.choice([1, 1, 1, 2, 3, 5, 7])
    while kv * group > most:
        kv, group = max(1, kv // 2), max(1, group - 2)
    return kv * group, kv


# Limits of a drawn case: algorithmic flops well below the largest listed case's (small and ragged sizes run at a lower rate)
_MOST_FLOPS = {"train": 6e12, "forward": 3e12, "attention": 1.2e12}


def draw(rng):
    kind = rng.choice(["train", "train", "train", "train", "forward", "attention", "attention", "rows"])
    while True:
        if kind == "rows":
            return dict(kind=kind, rows=_log_int(rng, 128, 16384, 1), width=_log_int(rng, 256, 8192, 8))
        if kind == "attention":
            n, nk = _heads(rng, 16)
            case = dict(kind=kind, heads=n, kv_heads=nk, head_dim=rng.choice([64, 128, 128]), seq=_log_int(rng, 128, 16384, 8),
                        mbsz=rng.choice([1, 1, 2, 4, 8]), causal=rng.random() < 0.7)
            if case["seq"] * case["mbsz"] > 32768:
                continue
        elif kind == "train" and rng.random() < 0.15:      # the fp32 configuration's range
            n, nk = _heads(rng, 4)
            case = dict(kind=kind, layers=1, microbatches=rng.choice([2, 3]), serial=rng.random() < 0.3,
                        **_layer(_log_int(rng, 64, 512, 8), n, nk, rng.choice([32, 64]), _log_int(rng, 128, 1024, 8), _log_int(rng, 40, 256, 8),
                                 1, rng.choice([1, 2, 4]), dtype="f32", **rng.choice([_GPT, _LLAMA])))
        else:
            n, nk = _heads(rng, 16)
            step = rng.choice([8, 32, 128])
            options = dict(rng.choice([_GPT, _LLAMA]), causal=rng.random() < 0.8)
            case = dict(kind=kind, layers=rng.choice([1, 1, 2]),
                        **_layer(_log_int(rng, 512, 7168, step), n, nk, rng.choice([64, 128, 128]), _log_int(rng, 512, 8192, step),
                                 _log_int(rng, 256, 6144, 8), rng.choice([1, 1, 2, 3]), rng.choice([1, 2, 4, 8]), **options))
            if kind == "train":
                case.update(microbatches=rng.choice([2, 3, 4]), serial=rng.random() < 0.3)
            if case["seq"] * case["mbsz"] > 12288:
                continue
        if work(case)["flops"] <= _MOST_FLOPS[kind]:
            return case


# ---- what one pass cannot do without -------------------------------------------------------------------------------

def _dims(c):
    T, d = c["seq"] * c["mbsz"], c["head_dim"]
    a, q = c["heads"] * d, (c["heads"] + 2 * c["kv_heads"]) * d
    pairs = c["mbsz"] * (c["seq"] * (c["seq"] + 1) // 2 if c["causal"] else c["seq"] * c["seq"])
    return T, a, q, 4 * a * pairs          # tokens, widths of the attention output and of QKV, flops of the two attention products


def work(case):
    c = case
    if c["kind"] == "rows":
        n = c["rows"] * c["width"]
        # norm forward 2 tensors, backward 4 (x, dy, residual -> dx); GELU 2 + 3; SwiGLU 3 + 5; softmax 2 + 3; column sum 1
        return {"bytes": 25 * n * 2, "flops": 0}
    T, a, q, att = _dims(c)
    if c["kind"] == "attention":
        return {"bytes": (T * q * 2 + T * a * 2) * 2, "flops": 3 * att}     # qkv, dctx in; ctx, dqkv out
    es = 2 if c["dtype"] == "bf16" else 4
    h, f = c["hidden"], c["ffn"]
    weights = h * q + a * h + (3 if c["act"] == "swiglu" else 2) * h * f
    gemm = 2 * T * weights
    if c["kind"] == "forward":
        return {"bytes": c["layers"] * weights * es + 2 * T * h * es, "flops": c["layers"] * (gemm + att)}
    mb = c["microbatches"]
    # weights in, fp32 weight gradients out; per microbatch X and dY in, Y and dX out.  Backward: the gradient GEMMs
    # cost the forward's flops twice, attention four products for the forward's two
    return {"bytes": c["layers"] * weights * (es + 4) + mb * 4 * T * h * es, "flops": mb * c["layers"] * (3 * gemm + 3 * att)}


def tolerance(case):
    """Measured against plain fp32 / fp64 references of the same inputs (2-norm over an output, the worst output of the
    listed cases): fp32 layers 7e-7, the row kernels 1.7e-3, attention 2.4e-3 and whole bf16 layers, which chain up to a
    dozen rounded intermediates per layer, 5e-3 to 1.15e-2; stated about four times as large (layers: three times)."""
    if case["kind"] == "rows":
        return {"rel": 0.007}
    if case["kind"] == "attention":
        return {"rel": 0.01}
    return {"rel": 0.035 if case["dtype"] == "bf16" else 4e-6}


# ---- inputs and state ----------------------------------------------------------------------------------------------

_streams = None


def _side_streams():
    """The three streams of the program (made once, used by every stage)."""
    global _streams
    if _streams is None:
        _streams = [torch.cuda.Stream() for _ in range(3)]
    return _streams


class _Draws:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = dtype

    def normal(self, shape, std=1.0, mean=0.0):
        x = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=self.g)
        return x.to(self.dtype)


def _workload(c):
    return Workload("case", c["hidden"], c["heads"], c["head_dim"], c["ffn"], c["seq"], c["tp"], dtype=c["dtype"], norm=c["norm"],
                    act=c["act"], causal=c["causal"], rope=c["rope"], has_bias=c["has_bias"], kv_heads=c["kv_heads"])


def _weights(c, draws):
    """One layer's weights: matrices and biases N(0, 0.02) (narrower beyond hidden 4096, so that the pre-activations
    keep their scale), norm gains 1 + N(0, 0.02), norm biases N(0, 0.02)."""
    h, f, d = c["hidden"], c["ffn"], c["head_dim"]
    a, q = c["heads"] * d, (c["heads"] + 2 * c["kv_heads"]) * d
    std = 0.02 * min(1.0, math.sqrt(4096 / h))
    shapes = {"norm1_g": (h,), "w_qkv": (h, q), "w_o": (a, h), "norm2_g": (h,), "w_fc1": (h, f), "w_fc2": (f, h)}
    if c["norm"] == "ln":
        shapes.update(norm1_b=(h,), norm2_b=(h,))
    if c["act"] == "swiglu":
        shapes["w_up"] = (h, f)
    if c["has_bias"]:
        shapes.update(b_qkv=(q,), b_o=(h,), b_fc1=(f,), b_fc2=(h,))
    out = {}
    for key, shape in shapes.items():
        gain = key in ("norm1_g", "norm2_g")
        out[key] = draws.normal(shape, 0.02 if key.startswith("norm") else std, 1.0 if gain else 0.0)
    return out


def _pointers(table, tensors):
    return table(**{k: v.data_ptr() for k, v in tensors.items()})


def _prepare_train(c, seed):
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    draws = _Draws(seed, dtype)
    L, M, T = c["layers"], c["microbatches"], c["seq"] * c["mbsz"]
    ctx = stp.Context(torch.cuda.current_device())
    descs = (B.LayerDesc * L)(*[stp.make_desc(_workload(c), mbsz=c["mbsz"]) for _ in range(L)])
    weights = [_weights(c, draws) for _ in range(L)]
    # the gradient accumulators of the stage are one block of memory, so that clearing them is one fill
    flat = torch.zeros(sum(v.numel() for w in weights for v in w.values()), dtype=torch.float32, device="cuda")
    grads, at = [], 0
    for w in weights:
        g = {}
        for k, v in w.items():
            g[k] = flat[at:at + v.numel()].view(v.shape)
            at += v.numel()
        grads.append(g)
    nbytes = ctx.stash_bytes(descs[0])
    stash = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for _ in range(L * M)]
    act = [draws.normal((T, c["hidden"])) if i < M else torch.empty((T, c["hidden"]), dtype=dtype, device="cuda") for i in range((L + 1) * M)]
    grad = [draws.normal((T, c["hidden"])) if i >= L * M else torch.empty((T, c["hidden"]), dtype=dtype, device="cuda")
            for i in range((L + 1) * M)]
    tables = dict(w=(B.Weights * L)(*[_pointers(B.Weights, w) for w in weights]), g=(B.WGrads * L)(*[_pointers(B.WGrads, g) for g in grads]),
                  stash=(B.Stash * (L * M))(*[B.Stash(base=m.data_ptr(), bytes=nbytes) for m in stash]),
                  act=(C.c_void_p * ((L + 1) * M))(*[t.data_ptr() for t in act]),
                  grad=(C.c_void_p * ((L + 1) * M))(*[t.data_ptr() for t in grad]))
    ctx.ensure_workspace(list(descs))
    steps = [(B.Op * len(s))(*s) for s in S.stage_sequence(L, M)]
    outputs = {"y": act[L * M:], "dx": grad[:M], "dw": grads}
    return dict(kind="train", ctx=ctx, stage=B.Stage(n_layers=L, n_microbatches=M, desc=descs, **tables), steps=steps, flat=flat,
                serial=c["serial"], outputs=outputs, keep=(descs, weights, tables, stash, act, grad))


def _run_train(s):
    ctx, now = s["ctx"], torch.cuda.current_stream()
    s["flat"].zero_()
    streams = [now] * 3 if s["serial"] else _side_streams()
    if not s["serial"]:
        for q in streams:
            q.wait_stream(now)
    ctx.braid_reset()
    for ops in s["steps"]:
        ctx.braid_step(s["stage"], ops, *streams)
    if not s["serial"]:
        for q in streams:
            now.wait_stream(q)
    return s["outputs"]


def _prepare_forward(c, seed):
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    draws = _Draws(seed, dtype)
    T = c["seq"] * c["mbsz"]
    ctx = stp.Context(torch.cuda.current_device())
    desc = stp.make_desc(_workload(c), mbsz=c["mbsz"])
    weights = [_weights(c, draws) for _ in range(c["layers"])]
    nbytes = ctx.stash_bytes(desc)
    mem = torch.empty(nbytes, dtype=torch.uint8, device="cuda")        # no backward pass follows: the layers share one stash
    x = [draws.normal((T, c["hidden"]))] + [torch.empty((T, c["hidden"]), dtype=dtype, device="cuda") for _ in range(c["layers"])]
    ctx.ensure_workspace([desc])
    return dict(kind="forward", ctx=ctx, desc=desc, w=[_pointers(B.Weights, w) for w in weights], stash=B.Stash(base=mem.data_ptr(), bytes=nbytes),
                x=x, mid=torch.empty_like(x[0]), keep=(weights, mem))


def _run_forward(s):
    ctx, desc, stash, now = s["ctx"], s["desc"], s["stash"], torch.cuda.current_stream()
    for l, w in enumerate(s["w"]):
        x, mid, y = s["x"][l], s["mid"], s["x"][l + 1]
        ctx.forward_unit(desc, B.PRE_ATTN, w, stash, x_in=x, stream=now)
        ctx.forward_unit(desc, B.ATTN, w, stash, x_resid=x, y_out=mid, stream=now)
        ctx.forward_unit(desc, B.PRE_MLP, w, stash, x_in=mid, stream=now)
        ctx.forward_unit(desc, B.MLP, w, stash, x_resid=mid, y_out=y, stream=now)
    return s["x"][-1]


def _prepare_attention(c, seed):
    draws = _Draws(seed, torch.bfloat16)
    T, a, q, _ = _dims(c)
    ctx = stp.Context(torch.cuda.current_device())
    wl = Workload("case", 1024, c["heads"], c["head_dim"], 1024, c["seq"], 1, causal=c["causal"], kv_heads=c["kv_heads"])
    desc = stp.make_desc(wl, mbsz=c["mbsz"])
    ctx.ensure_workspace([desc])
    rows = c["mbsz"] * c["heads"] * c["seq"]
    return dict(kind="attention", ctx=ctx, desc=desc, qkv=draws.normal((T, q)), dout=draws.normal((T, a)),
                out=torch.empty((T, a), dtype=torch.bfloat16, device="cuda"), lse=torch.empty(rows, dtype=torch.float32, device="cuda"),
                delta=torch.empty(rows, dtype=torch.float32, device="cuda"), dqkv=torch.empty((T, q), dtype=torch.bfloat16, device="cuda"))


def _run_attention(s):
    now = torch.cuda.current_stream()
    s["ctx"].attention_forward(s["desc"], s["qkv"], s["out"], s["lse"], stream=now)
    s["ctx"].attention_backward(s["desc"], s["qkv"], s["out"], s["lse"], s["dout"], s["delta"], s["dqkv"], stream=now)
    return {"out": s["out"], "lse": s["lse"], "dqkv": s["dqkv"]}


def _prepare_rows(c, seed):
    draws = _Draws(seed, torch.bfloat16)
    T, h = c["rows"], c["width"]
    ctx = stp.Context(torch.cuda.current_device())
    wl = Workload("case", h, 1, 64, h, (T + 7) // 8 * 8, 1)
    ctx.ensure_workspace([stp.make_desc(wl)])
    s = dict(kind="rows", ctx=ctx, T=T, h=h, gain=draws.normal((h,), 0.02, 1.0), bias=draws.normal((h,), 0.02),
             stats=torch.empty((T, 2), dtype=torch.float32, device="cuda"), sums=torch.zeros((4, h), dtype=torch.float32, device="cuda"))
    for k in ("x", "up", "dy", "resid"):
        s[k] = draws.normal((T, h))
    for k in ("norm", "dnorm", "gelu", "dgelu", "swiglu", "dgate", "dup", "softmax", "dsoftmax"):
        s[k] = torch.empty((T, h), dtype=torch.bfloat16, device="cuda")
    return s


def _run_rows(s):
    ctx, T, h, now = s["ctx"], s["T"], s["h"], torch.cuda.current_stream()
    n, bf = T * h, stp.BF16
    s["sums"].zero_()
    dgain, dbias, dresid, dcol = s["sums"]
    ctx.norm_forward(bf, stp.NORM_LN, T, h, 1e-5, s["x"], s["gain"], s["bias"], s["norm"], s["stats"], stream=now)
    ctx.norm_backward(bf, stp.NORM_LN, T, h, s["x"], s["gain"], s["stats"], s["dy"], s["resid"], s["dnorm"], dgain, dbias, stream=now,
                      d_resid_sum=dresid, d_resid_sum_scale=0.125)
    ctx.gelu_forward(bf, n, s["x"], s["gelu"], stream=now)
    ctx.gelu_backward(bf, n, s["x"], s["dy"], s["dgelu"], stream=now)
    ctx.swiglu_forward(bf, n, s["x"], s["up"], s["swiglu"], stream=now)
    ctx.swiglu_backward(bf, n, s["x"], s["up"], s["dy"], s["dgate"], s["dup"], stream=now)
    ctx.softmax_forward(bf, T, h, 1.0, False, s["x"], s["softmax"], stream=now)
    ctx.softmax_backward(bf, T, h, 1.0, s["softmax"], s["dy"], s["dsoftmax"], stream=now)
    ctx.colsum(bf, T, h, s["dy"], 1.0, dcol, stream=now)
    return {k: s[k] for k in ("norm", "dnorm", "gelu", "dgelu", "swiglu", "dgate", "dup", "softmax", "dsoftmax", "sums")}


def prepare(case, seed):
    return {"train": _prepare_train, "forward": _prepare_forward, "attention": _prepare_attention, "rows": _prepare_rows}[case["kind"]](case, seed)


def run(state):
    return {"train": _run_train, "forward": _run_forward, "attention": _run_attention, "rows": _run_rows}[state["kind"]](state)
