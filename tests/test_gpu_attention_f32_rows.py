"""fp32 attention: what a query may not see does not reach it, not even as 0 * inf or 0 * NaN; and as many (head, sequence)
pairs as there may be; and sequences of few rows, which have kernels and workgroups of their own."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from harness import rel_err, to_host


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def attention(ctx, n, nk, d, seq, mbsz, causal, qkv, dout):
    desc = stp.make_desc(Workload("w", 64, n, d, 64, seq, 1, dtype="f32", causal=causal, kv_heads=nk), mbsz=mbsz)
    out, dqkv = torch.zeros_like(dout), torch.zeros_like(qkv)
    lse, delta = (torch.zeros((mbsz, n, seq), device="cuda") for _ in range(2))
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)
    torch.cuda.synchronize()
    a, ak = n * d, nk * d
    return {"out": out, "lse": lse[0].t(), "dq": dqkv[:, :a], "dk": dqkv[:, a:a + ak], "dv": dqkv[:, a + ak:]}


# one head dimension per kernel instantiation; 168 rows: five blocks of 32 and one of eight; the row before the last block's
# end, its end, and one in the middle of a block
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("t", [45, 164, 167])
@pytest.mark.parametrize("n,nk,d", [(2, 2, 24), (4, 2, 64), (2, 1, 104)])
def test_rows_behind_the_causal_mask_stay_out(ctx, n, nk, d, t, bad):
    seq = 168
    g = torch.Generator(device="cuda").manual_seed(d)
    qkv = torch.randn((seq, (n + 2 * nk) * d), generator=g, device="cuda")
    dout = torch.randn((seq, n * d), generator=g, device="cuda")
    clean = attention(ctx, n, nk, d, seq, 1, True, qkv, dout)
    a, ak = n * d, nk * d
    before, after, others = slice(0, t), slice(t + 1, seq), [i for i in range(seq) if i != t]
    # the operand whose row t is replaced -> the rows of each result that do not depend on it
    untouched = {"q": {"out": others, "lse": others, "dq": others, "dk": after, "dv": after},
                 "k": {"out": before, "lse": before, "dq": before},
                 "v": {"out": before, "lse": slice(0, seq), "dq": before, "dv": slice(0, seq)},
                 "dout": {"out": slice(0, seq), "dq": others, "dk": after, "dv": after}}
    for operand, rows in untouched.items():
        x, y = qkv.clone(), dout.clone()
        if operand == "dout":
            y[t] = bad
        else:
            x[t, {"q": slice(0, a), "k": slice(a, a + ak), "v": slice(a + ak, None)}[operand]] = bad
        got = attention(ctx, n, nk, d, seq, 1, True, x, y)
        for name, r in rows.items():
            if clean[name][r].numel() == 0:     # no row behind the last one
                continue
            # rows computed one by one, or in blocks, each within 3e-6 of the exact value (fp32 sums in another order)
            assert rel_err(to_host(got[name][r]), to_host(clean[name][r])) < 6e-6, (operand, name)


def test_infinite_rows_keep_their_sign(ctx):
    """Every query sees every key: an infinite value is infinite in each output row, and an infinite upstream gradient
    in each value gradient, in the last, partly empty block as well."""
    n, d, seq = 2, 40, 72
    g = torch.Generator(device="cuda").manual_seed(1)
    qkv = torch.randn((seq, 3 * n * d), generator=g, device="cuda")
    dout = torch.randn((seq, n * d), generator=g, device="cuda")
    x, y = qkv.clone(), dout.clone()
    x[seq - 1, 2 * n * d:] = float("-inf")
    y[seq - 1] = float("inf")
    assert (attention(ctx, n, n, d, seq, 1, False, x, dout)["out"] == float("-inf")).all()
    assert (attention(ctx, n, n, d, seq, 1, False, qkv, y)["dv"] == float("inf")).all()


def launches(n, nk, d, seq, mbsz, causal):
    return stp.lib().stp_attn_bwd_f32_launches(C.byref(stp.make_desc(Workload("w", 64, n, d, 64, seq, 1, dtype="f32", causal=causal, kv_heads=nk), mbsz=mbsz)))


# the same among so many workgroups that row dot, dQ and dK / dV have a launch each; the sequences without the value keep their bits
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("t", [45, 167])
@pytest.mark.parametrize("n,nk,d", [(2, 2, 24), (4, 2, 64), (2, 1, 104)])
def test_rows_behind_the_causal_mask_stay_out_in_three_launches(ctx, n, nk, d, t, bad):
    seq = 168
    mbsz = 256 // (6 * (n + nk)) + 1
    assert launches(n, nk, d, seq, mbsz, True) == 3 and launches(n, nk, d, seq, 1, True) == 1
    g = torch.Generator(device="cuda").manual_seed(d)
    qkv = torch.randn((mbsz * seq, (n + 2 * nk) * d), generator=g, device="cuda")
    dout = torch.randn((mbsz * seq, n * d), generator=g, device="cuda")
    clean = attention(ctx, n, nk, d, seq, mbsz, True, qkv, dout)
    a, ak = n * d, nk * d
    before, after, others = slice(0, t), slice(t + 1, seq), [i for i in range(seq) if i != t]
    untouched = {"q": {"dq": others, "dk": after, "dv": after}, "k": {"dq": before}, "v": {"dq": before, "dv": slice(0, seq)},
                 "dout": {"dq": others, "dk": after, "dv": after}}
    for operand, rows in untouched.items():
        x, y = qkv.clone(), dout.clone()
        if operand == "dout":
            y[t] = bad
        else:
            x[t, {"q": slice(0, a), "k": slice(a, a + ak), "v": slice(a + ak, None)}[operand]] = bad
        got = attention(ctx, n, nk, d, seq, mbsz, True, x, y)
        for name in ("out", "dq", "dk", "dv"):
            assert torch.equal(got[name][seq:], clean[name][seq:]), (operand, name)
        for name, r in rows.items():
            if clean[name][:seq][r].numel():
                # as above: rows computed one by one, or in blocks, each within 3e-6 of the exact value
                assert rel_err(to_host(got[name][:seq][r]), to_host(clean[name][:seq][r])) < 6e-6, (operand, name)


def test_infinite_rows_keep_their_sign_in_three_launches(ctx):
    n, d, seq, mbsz = 2, 40, 72, 24
    assert launches(n, n, d, seq, mbsz, False) == 3
    g = torch.Generator(device="cuda").manual_seed(1)
    qkv = torch.randn((mbsz * seq, 3 * n * d), generator=g, device="cuda")
    y = torch.randn((mbsz * seq, n * d), generator=g, device="cuda")
    y[seq - 1] = float("inf")
    dv = attention(ctx, n, n, d, seq, mbsz, False, qkv, y)["dv"]
    assert (dv[:seq] == float("inf")).all() and dv[seq:].isfinite().all()


# more pairs than a grid's second or third dimension holds (65535), and more than 2^20
@pytest.mark.parametrize("n,nk,mbsz", [(8, 8, 8250), (64, 1, 16500)])
def test_many_pairs(ctx, n, nk, mbsz):
    d, seq = 8, 32
    g = torch.Generator(device="cuda").manual_seed(n)
    qkv = torch.randn((mbsz * seq, (n + 2 * nk) * d), generator=g, device="cuda")
    dout = torch.randn((mbsz * seq, n * d), generator=g, device="cuda")
    got = attention(ctx, n, nk, d, seq, mbsz, True, qkv, dout)
    for first in (0, 8190, mbsz - 4):              # the same sequences by themselves: the same sums, bit for bit
        rows = slice(first * seq, (first + 4) * seq)
        few = attention(ctx, n, nk, d, seq, 4, True, qkv[rows].contiguous(), dout[rows].contiguous())
        for name in ("out", "dq", "dk", "dv"):
            assert torch.equal(got[name][rows], few[name]), (name, first)


# a wave per row in all three kernels; in the backward ones, in dK / dV only; blocks with one, two and all waves a workgroup; with a
# group of heads dK / dV has several blocks where the others have one; the same sequences few and many at a time
@pytest.mark.parametrize("seq,mbsz,n,d,causal,nk", [(1, 8, 3, 64, True, 0), (5, 8, 2, 24, False, 0), (12, 2, 2, 64, True, 0), (20, 2, 1, 32, True, 0),
                                                    (24, 1, 2, 128, False, 0), (24, 1, 2, 16, True, 0), (32, 1, 8, 48, True, 1), (40, 1, 2, 64, False, 0),
                                                    (64, 1, 4, 104, True, 2), (72, 1, 2, 128, True, 0), (4, 130, 8, 64, True, 0), (8, 130, 8, 64, True, 0),
                                                    (8, 70, 8, 128, False, 1), (16, 40, 8, 40, True, 0)])
def test_few_rows(ctx, seq, mbsz, n, d, causal, nk):
    import test_gpu_kernels
    test_gpu_kernels.test_attention_forward_backward(ctx, "f32", seq, mbsz, n, d, causal, nk)


# few workgroups take row dot, dQ and dK / dV in one launch: at its limit of 256 of them (two blocks of a sequence, 2 * 64 heads), and the same
# sequences among more, where each has a launch of its own
@pytest.mark.parametrize("seq,n,nk,d,causal,mbsz", [(64, 64, 64, 64, True, 1), (128, 4, 4, 64, True, 1), (104, 2, 2, 24, False, 2), (200, 4, 2, 32, True, 1),
                                                    (96, 6, 2, 104, False, 1), (256, 8, 8, 128, True, 1), (48, 4, 4, 16, True, 1)])
def test_one_launch_has_the_bits_of_three(ctx, seq, n, nk, d, causal, mbsz):
    g = torch.Generator(device="cuda").manual_seed(seq)
    many = mbsz + 256 // (n + nk)
    assert (launches(n, nk, d, seq, mbsz, causal), launches(n, nk, d, seq, many, causal)) == (1, 3)
    qkv = torch.randn((many * seq, (n + 2 * nk) * d), generator=g, device="cuda")
    dout = torch.randn((many * seq, n * d), generator=g, device="cuda")
    few = attention(ctx, n, nk, d, seq, mbsz, causal, qkv[:mbsz * seq].contiguous(), dout[:mbsz * seq].contiguous())
    got = attention(ctx, n, nk, d, seq, many, causal, qkv, dout)
    for name in ("out", "dq", "dk", "dv"):
        assert torch.equal(got[name][:mbsz * seq], few[name]), name


def test_gradients_over_the_output(ctx):
    n, d, seq = 4, 64, 128
    g = torch.Generator(device="cuda").manual_seed(2)
    qkv, dout = (torch.randn((seq, w * n * d), generator=g, device="cuda") for w in (3, 1))
    want = attention(ctx, n, n, d, seq, 1, True, qkv, dout)
    desc = stp.make_desc(Workload("w", 64, n, d, 64, seq, 1, dtype="f32", causal=True, kv_heads=n))
    buf = torch.zeros((seq, 3 * n * d), device="cuda")
    out = buf.view(-1)[:seq * n * d].view(seq, n * d)
    lse, delta = (torch.zeros((1, n, seq), device="cuda") for _ in range(2))
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, buf)
    torch.cuda.synchronize()
    assert torch.equal(buf, torch.cat([want[k] for k in ("dq", "dk", "dv")], 1))


# one launch (to the limit of it, a partly empty block, groups of heads, rows computed one by one) and three
@pytest.mark.parametrize("seq,n,nk,d,causal,mbsz,bad", [(128, 4, 4, 64, True, 1, 0.0), (64, 64, 64, 64, True, 1, 0.0), (168, 2, 1, 104, False, 2, 0.0), (72, 8, 2, 24, True, 1, 0.0),
                                                        (128, 4, 4, 64, True, 1, float("nan")), (128, 64, 64, 32, True, 2, 0.0), (8, 4, 4, 64, True, 1, 0.0)])
def test_delta_is_the_row_sum(ctx, seq, n, nk, d, causal, mbsz, bad):
    g = torch.Generator(device="cuda").manual_seed(seq * n)
    qkv = torch.randn((mbsz * seq, (n + 2 * nk) * d), generator=g, device="cuda")
    dout = torch.randn((mbsz * seq, n * d), generator=g, device="cuda")
    if bad:
        dout[seq - 1] = bad
    desc = stp.make_desc(Workload("w", 64, n, d, 64, seq, 1, dtype="f32", causal=causal, kv_heads=nk), mbsz=mbsz)
    out, dqkv = torch.zeros_like(dout), torch.zeros_like(qkv)
    lse, delta = torch.zeros((mbsz, n, seq), device="cuda"), torch.full((mbsz, n, seq), 1e9, device="cuda")
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)
    torch.cuda.synchronize()
    terms = (dout.double() * out.double()).view(mbsz, seq, n, d).transpose(1, 2)
    want = terms.sum(-1)
    assert torch.equal(want.isnan(), delta.isnan())
    # d products and sums of 32 bits: at most d roundings of the sum of the terms' sizes
    assert ((delta.double() - want).abs() <= d * 2.0 ** -24 * terms.abs().sum(-1))[~want.isnan()].all()
