"""Attention forward at head dimension 64 with eight waves: one to a few steps of 128 keys, key blocks of which the second wave half sees
nothing, the mask's and the sequence's edges within a step, several chunks, groups of heads; in phase, and the few with the phases apart."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from test_gpu_kernels import test_attention_forward_backward as check


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    c.set_workspace(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"))
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("seq,mbsz,n,nk", [(8, 1, 1, 0), (64, 1, 2, 0), (72, 1, 2, 1), (128, 2, 1, 0), (136, 1, 3, 0), (192, 1, 2, 0), (200, 1, 2, 0),
                                           (264, 2, 2, 1), (320, 1, 4, 2), (520, 8, 8, 0), (392, 1, 1, 0), (312, 2, 2, 1), (184, 1, 3, 0), (1032, 1, 2, 0), (2056, 1, 1, 0)])
def test_edges(ctx, seq, mbsz, n, nk, causal):
    desc = stp.make_desc(Workload("w", 1024, n, 64, 1024, seq, 1, causal=causal, kv_heads=nk), mbsz=mbsz)
    apart, four = not causal and seq in (136, 184, 264, 312), not causal and mbsz == 8
    assert stp.lib().stp_attn_fwd_route(C.byref(desc)) == (1 if apart else 0 if four else 2)
    check(ctx, "bf16", seq, mbsz, n, 64, causal, nk)
