"""Attention backward in workgroups of four waves (head dimension 64, many short blocks) against an fp32 reference."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from harness import TOL, rel_err, to_host
from test_gpu_attention_routes import ctx, reference  # noqa: F401  (fixture)


# full blocks, blocks that end inside a tile, a half and a row; one block; grouped heads, whose key blocks run over the group; both masks
@pytest.mark.parametrize("n,nk,seq,mbsz,causal", [(8, 8, 520, 8, True), (16, 16, 256, 8, False), (16, 16, 128, 16, True), (16, 8, 200, 16, True),
                                                  (16, 16, 129, 16, True), (8, 8, 33, 64, False), (12, 12, 1000, 8, True), (16, 16, 8, 32, True)])
def test_against_fp32(ctx, n, nk, seq, mbsz, causal):  # noqa: F811
    desc = stp.make_desc(Workload("w", 1024, n, 64, 1024, seq, 1, causal=causal, kv_heads=nk), mbsz=mbsz)
    assert stp.lib().stp_attn_bwd_halves(C.byref(desc)) == 1
    ctx.ensure_workspace([desc])
    g = torch.Generator(device="cuda").manual_seed(n * seq + mbsz)
    T, a, width = seq * mbsz, n * 64, (n + 2 * nk) * 64
    qkv = torch.randn((T, width), generator=g, device="cuda").to(torch.bfloat16)
    dout = torch.randn((T, a), generator=g, device="cuda").to(torch.bfloat16)
    out = torch.empty((T, a), dtype=torch.bfloat16, device="cuda")
    dqkv = torch.full((T, width), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse, delta = (torch.empty((n * T,), device="cuda") for _ in range(2))
    ctx.attention_forward(desc, qkv, out, lse)
    ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)
    torch.cuda.synchronize()
    ref = reference(qkv, dout, n, nk, 64, seq, mbsz, causal)[2]
    for lo, hi in ((0, a), (a, a + nk * 64), (a + nk * 64, width)):
        assert rel_err(to_host(dqkv[:, lo:hi]), to_host(ref[:, lo:hi])) < TOL["bf16"]


# the exponentials among the MFMAs of dK / dV, or behind them where more workgroups follow than the chip holds at once: the same sums either way.  Blocks
# that end inside a tile, a half and a row, groups of heads, both masks
@pytest.mark.parametrize("n,nk,seq,few,many,causal", [(16, 16, 40, 16, 24, False), (12, 12, 136, 10, 16, True), (16, 8, 200, 10, 16, False), (8, 8, 264, 10, 16, True),
                                                      (12, 12, 520, 4, 8, False)])
def test_one_round_has_the_bits_of_several(ctx, n, nk, seq, few, many, causal):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(seq)
    T, a, width = seq * many, n * 64, (n + 2 * nk) * 64
    qkv = torch.randn((T, width), generator=g, device="cuda").to(torch.bfloat16)
    dout = torch.randn((T, a), generator=g, device="cuda").to(torch.bfloat16)
    out, lse = torch.randn((T, a), generator=g, device="cuda").to(torch.bfloat16), torch.rand((many * n * seq,), generator=g, device="cuda") + 4.0
    got = []
    for mbsz, among in ((few, 1), (many, 0)):
        desc = stp.make_desc(Workload("w", 1024, n, 64, 1024, seq, 1, causal=causal, kv_heads=nk), mbsz=mbsz)
        assert stp.lib().stp_attn_bwd_halves(C.byref(desc)) == 1 and stp.lib().stp_attn_bwd_between(C.byref(desc)) == among
        ctx.ensure_workspace([desc])
        dqkv, delta = torch.full((seq * mbsz, width), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.empty_like(lse)
        ctx.attention_backward(desc, qkv, out, lse, dout, delta, dqkv)       # any output and log-sum-exp will do
        got.append(dqkv)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1][:seq * few])
