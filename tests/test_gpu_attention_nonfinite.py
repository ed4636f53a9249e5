"""NaN and infinities in the bf16 attention: they reach the rows that depend on them, and no other sequence, no row that the mask keeps from a key of that
value, no row before the tile in which masked rows are multiplied by zero.  Each route of the forward and of the backward."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from test_gpu_attention_routes import ctx  # noqa: F401  (fixture)

# heads, kv heads, head dimension, tokens, sequences, mask; routes of forward (0: four waves, 1: phases apart, 2: in phase) and backward (wave halves,
# exponentials among the MFMAs)
SHAPES = [(2, 1, 64, 392, 2, True, 2, 2, 1), (2, 1, 128, 392, 2, True, 1, 2, 0), (12, 12, 64, 264, 6, True, 2, 1, 1), (16, 16, 64, 264, 8, True, 0, 1, 0),
          (4, 4, 64, 136, 2, False, 1, 2, 1)]


def run(ctx, desc, qkv, dout):  # noqa: F811
    out, dqkv = torch.empty_like(dout), torch.empty_like(qkv)
    lse, delta = (torch.empty((desc.mbsz, desc.heads_local, desc.seq), device="cuda") for _ in range(2))
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)
    torch.cuda.synchronize()
    a, ak, d = dout.shape[1], (qkv.shape[1] - dout.shape[1]) // 2, desc.head_dim
    rows = lambda t: t.reshape(desc.mbsz, desc.seq, -1, d)  # noqa: E731
    return {"out": rows(out), "dq": rows(dqkv[:, :a]), "dk": rows(dqkv[:, a:a + ak]), "dv": rows(dqkv[:, a + ak:]), "lse": lse.transpose(1, 2)[..., None]}


@pytest.mark.parametrize("n,nk,d,seq,mbsz,causal,fwd,halves,among", SHAPES)
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("t", [5, 130])
def test_reach(ctx, n, nk, d, seq, mbsz, causal, fwd, halves, among, bad, t):  # noqa: F811
    desc = stp.make_desc(Workload("w", 1024, n, d, 1024, seq, 1, causal=causal, kv_heads=nk), mbsz=mbsz)
    L = stp.lib()
    assert (L.stp_attn_fwd_route(C.byref(desc)), L.stp_attn_bwd_halves(C.byref(desc)), L.stp_attn_bwd_between(C.byref(desc))) == (fwd, halves, among)
    ctx.ensure_workspace([desc])
    g = torch.Generator(device="cuda").manual_seed(seq + d)
    qkv = torch.randn((mbsz * seq, (n + 2 * nk) * d), generator=g, device="cuda").to(torch.bfloat16)
    dout = torch.randn((mbsz * seq, n * d), generator=g, device="cuda").to(torch.bfloat16)
    clean = run(ctx, desc, qkv, dout)
    assert all(x.isfinite().all() for x in clean.values())
    a, ak, block = n * d, nk * d, t // 128 * 128
    every, none = slice(0, seq), slice(0, 0)
    before, others, after = (slice(0, t), [i for i in range(seq) if i != t], slice(block + 128, seq)) if causal else (none, [i for i in range(seq) if i != t], none)
    sees, seen = (slice(t, seq), slice(0, t + 1)) if causal else (every, every)
    early = slice(0, block) if causal else none
    # the operand whose row t is replaced -> rows of each result that do not depend on it, rows that do
    cases = {"q": ({"out": others, "lse": others, "dq": others, "dk": after, "dv": after}, {"out": [t], "dq": [t], "dk": seen, "dv": seen}),
             "k": ({"out": before, "lse": before, "dq": early}, {"out": sees, "dq": sees}),
             "v": ({"out": early, "lse": every, "dq": early}, {"out": sees, "dq": sees}),
             "dout": ({"out": every, "lse": every, "dq": others, "dk": after, "dv": after}, {"dq": [t], "dk": seen, "dv": seen})}
    for operand, (untouched, reached) in cases.items():
        x, y = qkv.clone(), dout.clone()
        if operand == "dout":
            y[t] = bad
        else:
            x[t, {"q": slice(0, a), "k": slice(a, a + ak), "v": slice(a + ak, None)}[operand]] = bad
        got = run(ctx, desc, x, y)
        for name in got:
            assert torch.equal(got[name][1:], clean[name][1:]), (operand, name, "other sequences")
        for name, r in untouched.items():
            assert torch.equal(got[name][0, r], clean[name][0, r]), (operand, name)
        if bad != bad:
            for name, r in reached.items():
                assert got[name][0, r].isnan().all(), (operand, name)
