"""Routes of the bf16 attention plan against an fp32 reference: four-wave forward workgroups (head dimension 64, many short
blocks), backward launches whose dq rows repeat once per query head of a group, blocks of one chunk beside blocks of several."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from harness import TOL, rel_err, to_host


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def reference(qkv, dout, n, nk, d, seq, mbsz, causal):
    x = qkv.float().view(mbsz, seq, n + 2 * nk, d).requires_grad_()
    q, k, v = x[:, :, :n], x[:, :, n:n + nk], x[:, :, n + nk:]
    k, v = (t.repeat_interleave(n // nk, dim=2) for t in (k, v))
    q, k, v = (t.transpose(1, 2).contiguous() for t in (q, k, v))
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) / d ** 0.5
    if causal:
        s = s.masked_fill(torch.ones(seq, seq, dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    out = torch.matmul(torch.softmax(s, dim=-1), v).transpose(1, 2).reshape(mbsz * seq, n * d)
    out.backward(dout.float())
    return out.detach(), torch.logsumexp(s.detach(), dim=-1).flatten(), x.grad.view(mbsz * seq, -1)


# forward: 0 four waves a workgroup, 1 eight with the phases apart, 2 eight in phase; backward: wave halves
@pytest.mark.parametrize("n,nk,d,seq,mbsz,causal,forward,backward", [
    (8, 8, 64, 520, 8, True, 2, 1),        # four waves in the backward; the last block has 8 rows
    (16, 16, 64, 520, 8, True, 0, 1),      # four waves in both
    (16, 16, 64, 72, 8, False, 2, 2),      # one block of 72 keys: one full tile, one of eight keys
    (16, 4, 64, 1000, 4, True, 0, 2),      # four waves in the forward, grouped heads
    (6, 2, 64, 1000, 3, True, 2, 2),       # key blocks of several chunks, query blocks of one
    (12, 4, 64, 776, 1, False, 2, 2),
    (6, 3, 64, 272, 2, False, 1, 2),       # phases apart, grouped heads
    (7, 1, 128, 1504, 1, True, 1, 2),      # seven dq rows per item
    (3, 1, 64, 4096, 1, True, 2, 2),       # chunks in all three kernels
    (10, 2, 128, 200, 2, True, 1, 2),
    (1, 1, 128, 2056, 1, False, 1, 2),
])
def test_against_fp32(ctx, n, nk, d, seq, mbsz, causal, forward, backward):
    g = torch.Generator(device="cuda").manual_seed(n * seq + mbsz)
    T, width = seq * mbsz, (n + 2 * nk) * d
    qkv = torch.randn((T, width), generator=g, device="cuda").to(torch.bfloat16)
    dout = torch.randn((T, n * d), generator=g, device="cuda").to(torch.bfloat16)
    desc = stp.make_desc(Workload("w", 1024, n, d, 1024, seq, 1, causal=causal, kv_heads=nk), mbsz=mbsz)
    assert (stp.lib().stp_attn_fwd_route(C.byref(desc)), stp.lib().stp_attn_bwd_halves(C.byref(desc))) == (forward, backward)
    ctx.ensure_workspace([desc])
    out = torch.full((T, n * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dqkv = torch.full((T, width), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse, delta = (torch.full((n * T,), float("nan"), device="cuda") for _ in range(2))
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)
    torch.cuda.synchronize()
    ref_out, ref_lse, ref_dqkv = reference(qkv, dout, n, nk, d, seq, mbsz, causal)
    assert rel_err(to_host(out), to_host(ref_out)) < TOL["bf16"]
    assert rel_err(to_host(lse), to_host(ref_lse)) < 1e-4        # fp32 sums of bf16-rounded products' exponentials
    a = n * d
    for lo, hi in ((0, a), (a, a + nk * d), (a + nk * d, width)):
        assert rel_err(to_host(dqkv[:, lo:hi]), to_host(ref_dqkv[:, lo:hi])) < TOL["bf16"]
